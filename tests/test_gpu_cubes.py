"""GPU checks of the two sweeps on LDS cubes, the default of small levels:
bitwise equal to separate sweeps in gmg_smooth, V-cycles (with the coarse
correction folded in) and solves, where cubes can go wrong: sizes around
multiples of the cube's eight cells, single planes and rows, odd sizes,
periodic directions shorter than the halo, inactive cells, every precision.
Separate sweeps are checked against the oracle in test_gpu_parity.py."""
import numpy as np
import pytest

from paper_2607_07687_amd import gmg as G
from paper_2607_07687_amd import problems as P
from tests.gpu_util import dev, require_gpu, rounded, say, torch
from tests.test_gpu_parity import STORE

pytestmark = pytest.mark.gpu

CASES = [((8, 8, 8), (False,) * 3), ((9, 7, 17), (False,) * 3), ((16, 24, 4), (True, True, True)),
         ((2, 40, 2), (True, False, True)), ((31, 1, 1), (False,) * 3), ((34, 18, 1), (False,) * 3),
         ((40, 30, 26), (False, True, False)), ((33, 20, 16), (False, True, True)),
         # whole cubes (the others are few enough for halves)
         ((64, 60, 56), (False, True, False)), ((65, 58, 60), (False,) * 3)]


@pytest.mark.parametrize("prec,storage", [("f32", "f32"), ("f32", "bf16"), ("f64", "f64")])
@pytest.mark.parametrize("n,per", CASES, ids=lambda c: "x".join(map(str, c)))
def test_cubes_match_separate_sweeps(n, per, prec, storage):
    require_gpu()
    say(f"cubes {n} {per} {prec}/{storage}")
    L, s, _ = P.random_problem(n, per, seed=sum(n), contrast=2.0, holes=0.1)
    dt = G.GMG_F64 if prec == "f64" else G.GMG_F32
    Ld, sd = dev(rounded(L, prec), prec), dev(rounded(s, prec), prec)
    # no tail: every level runs on cubes
    kw = dict(l_storage=STORE[storage], tail_cells=0, coarse_rtol=0.0)
    hc = G.gmg_setup(G.gmg_default_params(n, per, dt, **kw), Ld)
    hs = G.gmg_setup(G.gmg_default_params(n, per, dt, pair_sweeps=0, **kw), Ld)
    x0 = dev(np.random.default_rng(3).standard_normal(s.shape), prec)
    for sweeps in (2, 3, 4):
        xa, xb = x0.clone(), x0.clone()
        G.gmg_smooth(hc, 0, xa, sd, sweeps)
        G.gmg_smooth(hs, 0, xb, sd, sweeps)
        assert torch.equal(xa, xb)
    xa, xb = x0.clone(), x0.clone()
    G.gmg_vcycle(hc, xa, sd)
    G.gmg_vcycle(hs, xb, sd)
    assert torch.equal(xa, xb)
    xa.zero_()
    xb.zero_()
    ra, rb = G.gmg_solve(hc, xa, sd, 1e-5, 20), G.gmg_solve(hs, xb, sd, 1e-5, 20)
    assert torch.equal(xa, xb) and ra["history"] == rb["history"]
    hc.close()
    hs.close()
