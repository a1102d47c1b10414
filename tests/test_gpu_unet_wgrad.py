"""GPU checks of the tiled weight gradient at the edges of its tiles (octets
of voxels along w, chains of rows along h, shares of planes), in every channel
tiling and on channel views, against FP64 sums over the valid pairs of voxels;
and that a voxel at the grid's edge that holds an infinity reaches no tap it
has no pair for."""
import pytest

from paper_2607_07687_amd import unet as UN
from tests.gpu_util import require_gpu, say, torch

pytestmark = pytest.mark.gpu

# (n, d, h, w, cin, cout)
CASES = [(1, 1, 1, 1, 8, 16), (1, 3, 5, 7, 16, 16), (2, 2, 4, 8, 32, 32), (1, 5, 9, 9, 16, 32),
         (1, 4, 17, 31, 32, 16), (2, 6, 16, 33, 8, 16), (1, 40, 12, 40, 16, 16),
         (1, 3, 8, 16, 64, 48), (1, 9, 33, 64, 32, 32), (2, 5, 6, 20, 48, 64),
         (1, 2, 3, 130, 128, 128), (1, 70, 30, 50, 32, 32)]


def reference(x, dy, magnitude=False):
    """dW [cout][3][3][3][cin] and db in FP64 over the pairs inside the grid."""
    if magnitude:
        x, dy = x.abs(), dy.abs()
    D, H, W = x.shape[1:4]
    dw = torch.zeros(dy.shape[4], 3, 3, 3, x.shape[4], dtype=torch.float64, device=x.device)

    def rng(k, m):  # dy indices whose shifted voxel is in the grid
        return max(0, 1 - k), min(m, m + 1 - k)
    for kd in range(3):
        for kh in range(3):
            for kw in range(3):
                (a, b), (c, e), (f, g) = rng(kd, D), rng(kh, H), rng(kw, W)
                if a >= b or c >= e or f >= g:
                    continue
                ys = dy[:, a:b, c:e, f:g].reshape(-1, dy.shape[4])
                xs = x[:, a + kd - 1:b + kd - 1, c + kh - 1:e + kh - 1, f + kw - 1:g + kw - 1]
                dw[:, kd, kh, kw] = ys.t().contiguous() @ xs.reshape(-1, x.shape[4])
    return dw, dy.sum((0, 1, 2, 3))


def run(s, x, dy, xld, xoff):
    n, d, h, w, cin = x.shape
    cout = dy.shape[4]
    wide = torch.full((n, d, h, w, xld), float("nan"), dtype=torch.bfloat16, device=x.device)
    wide[..., xoff:xoff + cin] = x
    ws = torch.full((UN.unet_wgrad_workspace(s, cin, cout, 27) // 4,), float("nan"), device=x.device)
    dw = torch.empty(cout, 3, 3, 3, cin, device=x.device)
    db = torch.empty(cout, device=x.device)
    UN.unet_conv_wgrad(s, UN.act(wide, xld, xoff, cin), UN.act(dy, cout, 0, cout), 27, dw, db, ws)
    return dw, db


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_tiled_wgrad(case):
    require_gpu()
    n, d, h, w, cin, cout = case
    say(f"tiled wgrad {case}")
    g = torch.Generator(device="cuda").manual_seed(sum(case))
    x = torch.randn(n, d, h, w, cin, device="cuda", generator=g).to(torch.bfloat16)
    dy = torch.randn(n, d, h, w, cout, device="cuda", generator=g).to(torch.bfloat16)
    s = UN.shape(n, d, h, w)
    if cout == 48 and not UN.unet_wgrad_kernel(s, cin, cout, 27)["rows"]:
        pytest.skip("48 output channels are taken on regular grids only")
    dw, db = run(s, x, dy, cin + 16, 8)
    rw, rb = reference(x.double(), dy.double())
    mw, mb = reference(x.double(), dy.double(), magnitude=True)
    # exact products, FP32 sums of at most 256 terms in a row (a step's rows, a
    # share's steps, the shares): 256 half units in the last place of the sum
    # of magnitudes
    tol = 256 * 2.0 ** -24
    assert ((dw.double() - rw).abs() <= tol * mw).all()
    assert ((db.double() - rb).abs() <= tol * mb).all()

    # an infinity at the high corner, one at the low corner
    x[0, d - 1, h - 1, w - 1, 0] = float("inf")
    x[0, 0, 0, 0, cin - 1] = float("inf")
    dw, db = run(s, x, dy, cin + 16, 8)
    rw, rb = reference(x.double(), dy.double())
    assert torch.equal(dw.isfinite(), rw.isfinite()) and db.isfinite().all()
