"""GPU checks of the 3x3x3 convolution and its weight gradient on planes of 2^27
elements and more, where byte offsets within one plane or a few pass 2^31.  The
convolution: bitwise the results of slabs of rows, which are grids of small planes
(their kernels are checked against FP64 sums in test_gpu_unet_dispatch.py).  The
weight gradient: of a few voxels in zeros, against their FP64 sums."""
import pytest

from paper_2607_07687_amd import unet as UN
from tests.gpu_util import require_gpu, say, torch

pytestmark = pytest.mark.gpu

# (d, h, w, cin, cout): a plane of 2^27 elements (marching), three of 2^28 (bricks),
# three of 2^30 (marching) in every instance, one a little smaller (bricks)
CASES = [(1, 2048, 2048, 32, 16), (3, 2048, 2048, 64, 16), (3, 8192, 8192, 16, 16),
         (1, 8192, 16384, 8, 16), (1, 4096, 8192, 32, 16), (1, 8192, 8192, 16, 32),
         (1, 4000, 4096, 64, 32)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_large_planes_match_slabs(case):
    require_gpu()
    d, h, w, cin, cout = case
    say(f"large planes {case} {UN.unet_conv_launch(UN.shape(1, d, h, w), cin, cout, 27)}")
    g = torch.Generator(device="cuda").manual_seed(h + cin)
    x = torch.empty(d, h, w, cin, dtype=torch.bfloat16, device="cuda")
    for k in range(d):  # in pieces: the FP32 numbers take twice the room
        for a in range(0, h, 1024):
            x[k, a:a + 1024] = torch.randn(min(1024, h - a), w, cin, device="cuda", generator=g)
    wt = torch.randn(cout, 27, cin, device="cuda", generator=g).to(torch.bfloat16)
    bias = torch.randn(cout, device="cuda", generator=g)

    def conv(t):
        y = torch.empty(*t.shape[:3], cout, dtype=torch.bfloat16, device="cuda")
        s = UN.shape(1, *t.shape[:3])
        UN.unet_conv_fwd(s, UN.act(t, cin, 0, cin), wt, bias, 27, UN.act(y, cout, 0, cout), None, 1)
        return y
    y = conv(x)
    for a in (0, h // 3, h // 2 - 20, h - 40):  # the middle one about byte 2^30 of 2^31
        lo, hi = max(0, a - 1), min(h, a + 41)
        part = conv(x[:, lo:hi].contiguous())
        assert torch.equal(y[:, a:a + 40], part[:, a - lo:a - lo + 40]), a


# (d, h, w, cin, cout): planes of 2^30 elements of x or dy, in every instance
WGRAD = [(2, 8192, 8192, 16, 16), (1, 8192, 16384, 8, 16), (1, 8192, 8192, 16, 32),
         (1, 4096, 8192, 32, 16), (1, 4096, 8192, 32, 32)]


@pytest.mark.parametrize("case", WGRAD, ids=lambda c: "x".join(map(str, c)))
def test_large_planes_weight_gradient(case):
    require_gpu()
    d, h, w, cin, cout = case
    s = UN.shape(1, d, h, w)
    say(f"large planes wgrad {case} {UN.unet_wgrad_launch(s, cin, cout, 27)}")
    assert UN.unet_wgrad_launch(s, cin, cout, 27)[0][0] == "tiled"
    g = torch.Generator(device="cuda").manual_seed(w + cin)

    def pick(m, n):
        return torch.randint(0, m, (n,), device="cuda", generator=g)
    # voxels of dy: anywhere, and at the grid's corners; x next to each of them
    v = [torch.cat([pick(m, 300), torch.tensor([0, m - 1, 0, m - 1], device="cuda")])
         for m in (d, h, w)]
    x = torch.zeros(d, h, w, cin, dtype=torch.bfloat16, device="cuda")
    dy = torch.zeros(d, h, w, cout, dtype=torch.bfloat16, device="cuda")
    n = len(v[0])
    dy[v[0], v[1], v[2]] = torch.randn(n, cout, device="cuda", generator=g).to(torch.bfloat16)
    for _ in range(6):
        u = [(a + pick(3, n) - 1).clamp(0, m - 1) for a, m in zip(v, (d, h, w))]
        x[u[0], u[1], u[2]] = torch.randn(n, cin, device="cuda", generator=g).to(torch.bfloat16)
    ws = torch.empty(UN.unet_wgrad_workspace(s, cin, cout, 27) // 4, device="cuda")
    dw, db = torch.empty(cout, 27, cin, device="cuda"), torch.empty(cout, device="cuda")
    UN.unet_conv_wgrad(s, UN.act(x, cin, 0, cin), UN.act(dy, cout, 0, cout), 27, dw, db, ws)
    at = torch.unique(torch.stack(v), dim=1)  # a voxel picked twice counts once
    ys = dy[at[0], at[1], at[2]].double()
    want = torch.zeros(cout, 27, cin, dtype=torch.float64, device="cuda")
    mag = torch.zeros_like(want)
    for t in range(27):
        u = [at[0] + t // 9 - 1, at[1] + t // 3 % 3 - 1, at[2] + t % 3 - 1]
        ok = torch.ones(at.shape[1], dtype=torch.bool, device="cuda")
        for a, m in zip(u, (d, h, w)):
            ok &= (a >= 0) & (a < m)
        xs = x[u[0][ok], u[1][ok], u[2][ok]].double()
        want[:, t] = ys[ok].t().contiguous() @ xs
        mag[:, t] = ys[ok].abs().t().contiguous() @ xs.abs()
    # exact products of at most 304 voxels, each added once
    tol = 304 * 2.0 ** -24
    assert ((dw.double() - want).abs() <= tol * mag).all()
    assert ((db.double() - ys.sum(0)).abs() <= tol * ys.abs().sum(0)).all()
