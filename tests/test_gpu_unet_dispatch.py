"""GPU parity of every instance of the convolution kernels that a size can
choose (test_unet_dispatch.py checks on the host that the cases reach them all):
forward in FP32 and BF16, the gated data gradient where the channels allow one,
and the weight gradient, on ragged grids, against FP64 sums over the valid pairs
of voxels."""
import pytest

from paper_2607_07687_amd import unet as UN
from tests import test_gpu_unet_wgrad as WG
from tests.gpu_util import require_gpu, say, torch

pytestmark = pytest.mark.gpu

# (n, d, h, w, cin, cout)
CONV = [
    # bricks: rows x waves along d x waves along the channels, output blocks per wave
    (1, 4, 9, 19, 8, 16), (2, 5, 9, 17, 8, 128), (1, 35, 89, 17, 8, 16), (2, 55, 25, 17, 8, 32),
    (1, 4, 9, 18, 16, 16), (1, 22, 9, 18, 16, 64), (1, 9, 37, 17, 16, 128), (1, 54, 9, 17, 16, 128),
    (2, 5, 10, 17, 32, 128), (1, 4, 10, 17, 32, 16), (2, 11, 9, 17, 32, 128), (2, 43, 9, 19, 32, 32),
    (2, 45, 21, 17, 32, 16), (1, 4, 9, 17, 64, 32), (1, 4, 9, 17, 64, 16), (1, 45, 9, 17, 64, 64),
    (2, 44, 10, 17, 64, 32), (1, 4, 9, 17, 128, 32), (1, 4, 9, 17, 128, 16), (1, 22, 9, 17, 128, 64),
    (2, 34, 13, 17, 128, 32),
    # marching: several samples and tiles in a share, tiles reaching past the grid, one plane
    (2, 50, 154, 19, 8, 16), (2, 5, 151, 19, 16, 128), (2, 50, 153, 17, 16, 16),
    (2, 7, 133, 17, 32, 32), (3, 1, 200, 330, 8, 32), (3, 1, 200, 330, 16, 16),
    (3, 1, 200, 330, 16, 32), (3, 1, 200, 330, 32, 16),
    # gathered operands: grids one or two voxels wide
    (2, 229, 1, 1, 32, 128), (2, 149, 17, 1, 16, 128), (2, 26, 156, 1, 16, 128),
    (1, 163, 99, 1, 16, 128), (2, 223, 73, 1, 16, 128), (2, 43, 380, 2, 16, 128),
]

WGRAD = [
    # (input, output channels, octets along w) of a workgroup's tile
    (1, 8, 54, 43, 8, 16), (1, 5, 13, 29, 8, 16), (2, 5, 6, 70, 8, 32), (1, 5, 33, 15, 16, 16),
    (1, 5, 14, 30, 16, 16), (1, 7, 5, 75, 48, 16), (1, 5, 15, 9, 16, 32), (2, 5, 7, 30, 16, 32),
    (1, 5, 3, 70, 16, 64), (1, 20, 58, 6, 32, 16), (1, 6, 15, 14, 32, 16), (1, 6, 7, 30, 64, 16),
    (1, 24, 28, 135, 64, 64), (1, 11, 22, 6, 128, 64), (1, 6, 7, 14, 32, 32), (1, 6, 3, 30, 32, 64),
    # many tiles of few voxels
    (2, 160, 1, 1, 96, 64), (1, 127, 2, 1, 32, 32), (1, 1, 1, 4096, 16, 16), (1, 117, 1, 1, 8, 32),
    # voxel chunks
    (1, 6, 1, 1, 48, 128), (1, 2, 2, 2, 16, 16),
]


def reference(x, w, magnitude=False):
    """Sum over taps and channels of w [cout][27][cin] and x [n][d][h][w][cin], FP64."""
    if magnitude:
        x, w = x.abs(), w.abs()
    n, d, h, wd, cin = x.shape
    y = torch.zeros(n, d, h, wd, w.shape[0], dtype=torch.float64, device=x.device)
    for t in range(27):
        kd, kh, kw = t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1

        def rng(k, m):  # outputs whose shifted voxel is in the grid
            return max(0, -k), min(m, m - k)
        (a, b), (c, e), (f, g) = rng(kd, d), rng(kh, h), rng(kw, wd)
        if a >= b or c >= e or f >= g:
            continue
        xs = x[:, a + kd:b + kd, c + kh:e + kh, f + kw:g + kw].reshape(-1, cin)
        y[:, a:b, c:e, f:g] += (xs @ w[:, t].t().contiguous()).reshape(n, b - a, e - c, g - f, -1)
    return y


@pytest.mark.parametrize("case", CONV, ids=lambda c: "x".join(map(str, c)))
def test_conv_instances(case):
    require_gpu()
    n, d, h, w, cin, cout = case
    s = UN.shape(n, d, h, w)
    say(f"conv {case} {UN.unet_conv_launch(s, cin, cout, 27, cin + 16)}")
    g = torch.Generator(device="cuda").manual_seed(sum(case))
    wide = torch.full((n, d, h, w, cin + 16), float("nan"), dtype=torch.bfloat16, device="cuda")
    x = torch.randn(n, d, h, w, cin, device="cuda", generator=g).to(torch.bfloat16)
    wide[..., 8:8 + cin] = x
    wt = torch.randn(cout, 27, cin, device="cuda", generator=g).to(torch.bfloat16)
    bias = torch.randn(cout, device="cuda", generator=g)
    xa = UN.act(wide, cin + 16, 8, cin)
    yf = torch.empty(n, d, h, w, cout, device="cuda")
    UN.unet_conv_fwd(s, xa, wt, bias, 27, UN.act(None, cout, 0, cout), yf, 0)
    want = reference(x.double(), wt.double())
    mag = reference(x.double(), wt.double(), magnitude=True)
    # exact products; FP32 sums of K / 32 steps of 32 products and the bias, each
    # addition within half a unit in the last place of the sum of magnitudes
    tol = (27 * cin / 32 + 33) * 2.0 ** -24
    assert ((yf.double() - (want + bias)).abs() <= tol * (mag + bias.abs())).all()
    # BF16 rows with ReLU, in a slice of a wider row: the same sums, rounded
    yb = torch.full((n, d, h, w, cout + 16), 3.0, dtype=torch.bfloat16, device="cuda")
    UN.unet_conv_fwd(s, xa, wt, bias, 27, UN.act(yb, cout + 16, 8, cout), None, 1)
    assert torch.equal(yb[..., 8:8 + cout], yf.clamp(min=0).to(torch.bfloat16))
    assert (yb[..., :8] == 3.0).all() and (yb[..., 8 + cout:] == 3.0).all()
    if cin < 16:
        return
    # the same convolution as a data gradient with the ReLU backward of its output
    wl = wt.flip(1).permute(2, 1, 0).contiguous()  # layer weights [cin][27][cout]
    gate = torch.randn(n, d, h, w, cout, device="cuda", generator=g).to(torch.bfloat16)
    fl = torch.empty(cin * 27 * cout, dtype=torch.int16, device="cuda")
    dx = torch.full((n, d, h, w, cout), 3.0, dtype=torch.bfloat16, device="cuda")
    UN.unet_conv_dgrad_relu(s, xa, wl, 27, UN.act(gate, cout, 0, cout), UN.act(dx, cout, 0, cout),
                            fl)
    UN.unet_conv_fwd(s, xa, wt, None, 27, UN.act(None, cout, 0, cout), yf, 0)
    assert torch.equal(dx, torch.where(gate > 0, yf, 0.0).to(torch.bfloat16))


@pytest.mark.parametrize("case", WGRAD, ids=lambda c: "x".join(map(str, c)))
def test_wgrad_instances(case):
    require_gpu()
    n, d, h, w, cin, cout = case
    s = UN.shape(n, d, h, w)
    say(f"wgrad {case} {UN.unet_wgrad_launch(s, cin, cout, 27, cin + 16)}")
    g = torch.Generator(device="cuda").manual_seed(sum(case))
    x = torch.randn(n, d, h, w, cin, device="cuda", generator=g).to(torch.bfloat16)
    dy = torch.randn(n, d, h, w, cout, device="cuda", generator=g).to(torch.bfloat16)
    dw, db = WG.run(s, x, dy, cin + 16, 8)
    rw, rb = WG.reference(x.double(), dy.double())
    mw, mb = WG.reference(x.double(), dy.double(), magnitude=True)
    tol = 256 * 2.0 ** -24  # of the sums of magnitudes, as in test_gpu_unet_wgrad.py
    assert ((dw.double() - rw).abs() <= tol * mw).all()
    assert ((db.double() - rb).abs() <= tol * mb).all()
    # infinities at two corners reach only the taps that pair them with a voxel
    x[0, d - 1, h - 1, w - 1, 0] = float("inf")
    x[0, 0, 0, 0, cin - 1] = float("inf")
    dw, db = WG.run(s, x, dy, cin + 16, 8)
    rw, _ = WG.reference(x.double(), dy.double())
    assert torch.equal(dw.isfinite(), rw.isfinite()) and db.isfinite().all()


@pytest.mark.parametrize("cout", [48, 80, 96])
def test_odd_output_blocks_in_voxel_chunks(cout):
    # regular grids take any multiple of 16 output channels, also where the rows of
    # a tile are past a descriptor's reach
    require_gpu()
    n, d, h, w, cin, ld = 1, 1, 4, 4096, 16, 8192
    s = UN.shape(n, d, h, w)
    assert UN.unet_wgrad_launch(s, cin, cout, 27, ld)[0] == ("chunk",)
    g = torch.Generator(device="cuda").manual_seed(cout)
    x = torch.randn(n, d, h, w, cin, device="cuda", generator=g).to(torch.bfloat16)
    dy = torch.randn(n, d, h, w, cout, device="cuda", generator=g).to(torch.bfloat16)
    dw, db = WG.run(s, x, dy, ld, 8)
    rw, rb = WG.reference(x.double(), dy.double())
    mw, mb = WG.reference(x.double(), dy.double(), magnitude=True)
    tol = 256 * 2.0 ** -24
    assert ((dw.double() - rw).abs() <= tol * mw).all()
    assert ((db.double() - rb).abs() <= tol * mb).all()
