"""GPU checks of the marching convolution (layers of few channels on grids of
many planes): bitwise the brick kernel's results, which slabs of the same grid
with too few planes get, over ragged tiles, several samples in a share, channel
views, FP32 output and the gated data gradient.  The brick kernel is checked
against the oracle in test_gpu_unet_bricks.py."""
import pytest

from paper_2607_07687_amd import unet as UN
from tests.gpu_util import require_gpu, say, torch

pytestmark = pytest.mark.gpu

N, D, H, W = 2, 301, 18, 40  # 4 tiles of 32 x 16 voxels: 2408 planes for 256 CUs
SLAB = 43


def bits(shape, g):
    return torch.randn(*shape, device="cuda", generator=g).to(torch.bfloat16).view(torch.int16)


@pytest.mark.parametrize("cin,cout", [(8, 16), (8, 32), (16, 16), (16, 32), (16, 64), (32, 16),
                                      (32, 32)])
@pytest.mark.parametrize("f32", [False, True])
def test_march_matches_bricks(cin, cout, f32):
    require_gpu()
    say(f"march {cin} -> {cout} f32 {f32}")
    g = torch.Generator(device="cuda").manual_seed(cin + cout)
    x = bits((N, D, H, W, cin + 8), g)
    wt, bias = bits((cout, 27, cin), g), torch.randn(cout, device="cuda", generator=g)

    def conv(t):
        s = UN.shape(*t.shape[:4])
        dt = torch.float32 if f32 else torch.int16
        y = torch.full(tuple(t.shape[:4]) + (cout + 16,), 3, dtype=dt, device="cuda")
        v = UN.act(None if f32 else y, cout + 16, 8, cout)
        UN.unet_conv_fwd(s, UN.act(t, cin + 8, 8, cin), wt, bias, 27, v, y if f32 else None, 1)
        return y
    y = conv(x)
    for n in range(N):
        for a in range(0, D, SLAB):
            b = min(D, a + SLAB)
            lo, hi = max(0, a - 1), min(D, b + 1)
            part = conv(x[n:n + 1, lo:hi].contiguous())
            assert torch.equal(y[n, a:b], part[0, a - lo:b - lo]), (n, a)


@pytest.mark.parametrize("cin,cout", [(16, 16), (32, 16), (16, 32), (32, 32)])
def test_march_gate(cin, cout):
    require_gpu()
    say(f"march gate {cin} <- {cout}")
    g = torch.Generator(device="cuda").manual_seed(cin * cout)
    s = UN.shape(N, D, H, W)
    dyt, yt, wt = bits((N, D, H, W, cout), g), bits((N, D, H, W, cin), g), bits((cout, 27, cin), g)
    dy, y = UN.act(dyt, cout, 0, cout), UN.act(yt, cin, 0, cin)
    fl = torch.empty(cout * 27 * cin, dtype=torch.int16, device="cuda")
    a, b = (torch.zeros((N, D, H, W, cin), dtype=torch.int16, device="cuda") for _ in "ab")
    va, vb = UN.act(a, cin, 0, cin), UN.act(b, cin, 0, cin)
    UN.unet_conv_dgrad_relu(s, dy, wt, 27, y, va, fl)
    UN.unet_conv_dgrad(s, dy, wt, 27, vb, fl)
    UN.unet_relu_bwd(s, y, vb, vb)
    assert torch.equal(a, b)
