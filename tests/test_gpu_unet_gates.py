"""GPU checks of the backward ops that apply the ReLU backward of their output
in the same pass: bitwise the plain op followed by unet_relu_bwd, on channel
views, ragged grids, channel counts off the vector paths, and gates that hold
zeros of both signs, subnormals, infinities and NaNs."""
import pytest

from paper_2607_07687_amd import unet as UN
from tests.gpu_util import require_gpu, say, torch

pytestmark = pytest.mark.gpu


def bits(shape, g, special=False):
    t = torch.randn(*shape, device="cuda", generator=g).to(torch.bfloat16).view(torch.int16)
    if special:
        vals = torch.tensor([0, -0x8000, 1, -0x7FFF, 0x7F80, -0x80, 0x7FC0, -0x40], device="cuda",
                            dtype=torch.int16)
        pick = torch.randint(0, 16, shape, device="cuda", generator=g)
        t = torch.where(pick < 8, vals[pick.clamp(max=7)], t)
    return t


@pytest.mark.parametrize("n,d,h,w,cin,cout", [(1, 5, 7, 9, 16, 16), (2, 8, 8, 16, 32, 32),
                                              (1, 3, 18, 33, 16, 64), (1, 4, 4, 4, 128, 128)])
@pytest.mark.parametrize("taps", [27, 1])
def test_dgrad_gate(n, d, h, w, cin, cout, taps):
    require_gpu()
    say(f"dgrad gate {(n, d, h, w, cin, cout, taps)}")
    g = torch.Generator(device="cuda").manual_seed(5)
    s = UN.shape(n, d, h, w)
    dyt = bits((n, d, h, w, cout), g)
    dy = UN.act(dyt, cout, 0, cout)
    wt = bits((cout, taps, cin), g)
    yt = bits((n, d, h, w, cin + 8), g, special=True)
    y = UN.act(yt, cin + 8, 8, cin)
    fl = torch.empty(cout * taps * cin, dtype=torch.int16, device="cuda")
    a, b = (torch.full((n, d, h, w, 2 * cin), 77, dtype=torch.int16, device="cuda") for _ in "ab")
    va, vb = UN.act(a, 2 * cin, cin, cin), UN.act(b, 2 * cin, cin, cin)
    UN.unet_conv_dgrad_relu(s, dy, wt, taps, y, va, fl)
    UN.unet_conv_dgrad(s, dy, wt, taps, vb, fl)
    UN.unet_relu_bwd(s, y, vb, vb)
    assert torch.equal(a, b)


@pytest.mark.parametrize("c", [8, 12, 32])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_pool_up_and_head_gates(c, accumulate):
    require_gpu()
    say(f"gates c {c} accumulate {accumulate}")
    g = torch.Generator(device="cuda").manual_seed(c)
    n, d, h, w, ld = 2, 4, 6, 10, 40
    f, cs = UN.shape(n, d, h, w), UN.shape(n, d // 2, h // 2, w // 2)

    keep = []  # a view holds no reference to its tensor

    def view(s, special=False):
        t = bits((s.n, s.d, s.h, s.w, ld), g, special)
        keep.append(t)
        return t, UN.act(t, ld, 8, c)
    _, small = view(cs)
    _, large = view(f)
    _, yf = view(f, special=True)
    _, yc = view(cs, special=True)
    a, va = view(f)
    b = a.clone()
    vb = UN.act(b, ld, 8, c)
    UN.unet_pool_bwd_relu(f, small, yf, va, accumulate)
    UN.unet_pool_bwd(f, small, vb, accumulate)
    UN.unet_relu_bwd(f, yf, vb, vb)
    assert torch.equal(a, b)

    a, va = view(cs)
    b = a.clone()
    vb = UN.act(b, ld, 8, c)
    UN.unet_up_bwd_relu(cs, large, yc, va)
    UN.unet_up_bwd(cs, large, vb)
    UN.unet_relu_bwd(cs, yc, vb, vb)
    assert torch.equal(a, b)

    wt = torch.randn(c, device="cuda", generator=g)
    dy = torch.randn(n, d, h, w, device="cuda", generator=g)
    ws = torch.empty(UN.unet_head_workspace(f, c) // 4 + 1, device="cuda")
    out = []
    for fused in (True, False):
        t = torch.full((n, d, h, w, ld), 77, dtype=torch.int16, device="cuda")
        dx = UN.act(t, ld, 8, c)
        dw, db = torch.empty(c, device="cuda"), torch.empty(1, device="cuda")
        if fused:
            UN.unet_head_bwd_relu(f, large, wt, dy, dx, dw, db, ws)
        else:
            UN.unet_head_bwd(f, large, wt, dy, dx, dw, db, ws)
            UN.unet_relu_bwd(f, large, dx, dx)
        out.append((t, dw, db))
    assert all(torch.equal(p, q) for p, q in zip(*out))
