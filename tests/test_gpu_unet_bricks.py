"""GPU parity of the brick kernel of the 3x3x3 convolutions against the FP64
oracle at the sizes where bricks can go wrong: grids narrower than a brick,
one voxel more or less than whole bricks, single planes and rows, channel
counts of one to eight chunks, and outputs whose rows are not 16-byte aligned.

Tolerances as for the other convolution cases: FP32 outputs differ by the
accumulation order alone (K <= 27 * 256 products: 1e-5 relative), BF16 ones
also by their rounding (2^-8 per element)."""
import numpy as np
import pytest

from oracle import unet_oracle as UO
from paper_2607_07687_amd import unet as UN
from tests.gpu_util import require_gpu, say
from tests.test_gpu_unet_ops import bf16_to_f64, cf, cl, rel, to_dev_bf16, w_gpu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # chunks of 8, 16 and 32 channels; one voxel, one row, one plane
    (1, 8, 16, (1, 1, 1)), (1, 16, 16, (1, 1, 17)), (2, 32, 32, (1, 5, 16)), (1, 32, 16, (5, 1, 1)),
    # 8-wide bricks
    (1, 16, 32, (5, 9, 8)), (1, 32, 32, (4, 17, 7)), (1, 8, 32, (3, 8, 6)),
    # several chunks of each size, K split over waves or not
    (1, 24, 16, (2, 3, 18)), (1, 40, 32, (3, 7, 15)), (1, 48, 64, (3, 9, 15)),
    (1, 96, 32, (2, 9, 33)), (1, 64, 128, (3, 7, 13)), (1, 128, 64, (2, 8, 16)),
    (1, 256, 16, (2, 4, 9)),
]


@pytest.mark.parametrize("n,cin,cout,dhw", CASES)
def test_conv_bricks(n, cin, cout, dhw):
    require_gpu()
    say(f"conv bricks {n} {cin}->{cout} {dhw}")
    rng = np.random.default_rng(300 + cin + cout + sum(dhw))
    # x as a channel slice [8, 8 + cin) of a wider row whose other channels
    # must not be read
    xw = np.full((n,) + dhw + (cin + 16,), np.nan)
    xw[..., 8:8 + cin] = cl(rng.standard_normal((n, cin) + dhw))
    w = rng.standard_normal((cout, cin, 3, 3, 3)) / np.sqrt(27 * cin)
    b = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    xd, xw64 = to_dev_bf16(xw)
    x64 = cf(xw64[..., 8:8 + cin])
    wd, w64 = to_dev_bf16(w_gpu(w))
    w64o = w64.reshape(cout, 27, cin).transpose(0, 2, 1).reshape(cout, cin, 3, 3, 3)
    want = np.stack([UO.conv3d(x64[i], w64o, b.astype(np.float64)) for i in range(n)])
    s, bd = UN.shape(n, *dhw), torch.from_numpy(b).cuda()
    xa = UN.act(xd, cin + 16, 8, cin)
    yf = torch.full((n,) + dhw + (cout,), np.nan, dtype=torch.float32, device="cuda")
    UN.unet_conv_fwd(s, xa, wd, bd, 27, UN.act(None, cout, 0, cout), yf, 0)
    assert rel(cf(yf.cpu().numpy().astype(np.float64)), want) <= 1e-5
    # BF16 rows that start 4 bytes past a 16-byte boundary, in slice
    # [8, 8 + cout) of a wider row: the narrow stores, and nothing beside them
    ld, nv = cout + 16, n * dhw[0] * dhw[1] * dhw[2]
    buf = torch.full((nv * ld + 8,), 0x7FC0, dtype=torch.int16, device="cuda")
    UN.unet_conv_fwd(s, xa, wd, bd, 27, UN.act(buf[2:2 + nv * ld], ld, 8, cout), None, 1)
    raw = buf.cpu().numpy()
    rows = raw[2:2 + nv * ld].reshape((n,) + dhw + (ld,))
    keep = np.ones(ld, bool)
    keep[8:8 + cout] = False
    assert np.all(rows[..., keep] == 0x7FC0) and np.all(raw[[0, 1, -1]] == 0x7FC0)
    got = cf(bf16_to_f64(rows[..., 8:8 + cout].copy().view(np.uint16)))
    wr = np.maximum(want, 0.0)
    assert np.all(np.abs(got - wr) <= 2.0 ** -8 * np.abs(wr) + 1e-5 * np.abs(wr).max())


def test_conv_bricks_keep_infinities_local():
    # an infinite input reaches exactly the outputs within one voxel of it:
    # neither the padded taps of a K step nor a brick's halo spread it
    require_gpu()
    for cin in (8, 16, 32):
        x = torch.zeros((1, 6, 11, 20, cin), dtype=torch.bfloat16, device="cuda")
        x[0, 3, 5, 15, 1] = float("inf")
        w = torch.ones((16, 27, cin), dtype=torch.bfloat16, device="cuda")
        y = torch.zeros((1, 6, 11, 20, 16), dtype=torch.float32, device="cuda")
        UN.unet_conv_fwd(UN.shape(1, 6, 11, 20), UN.act(x, cin, 0, cin), w, None, 27,
                         UN.act(None, 16, 0, 16), y, 0)
        want = torch.zeros_like(y)
        want[0, 2:5, 4:7, 14:17] = float("inf")
        assert torch.equal(y, want)
