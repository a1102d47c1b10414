"""GPU checks of the coarse levels smoothed from registers by one workgroup:
V-cycles bitwise equal to the same cycle composed of the per-level calls
(grid kernels), at the edges of the pairs a wavefront and a workgroup hold,
odd x sizes, periodic directions of two cells, inactive cells, in
LDS and in global memory.  The coarsest-level rule's sweep counts are
checked against the oracle in test_gpu_coarse_rule.py."""
import numpy as np
import pytest

from paper_2607_07687_amd import gmg as G
from paper_2607_07687_amd import problems as P
from tests.gpu_util import dev, require_gpu, rounded, say, torch
from tests.test_gpu_parity import STORE

pytestmark = pytest.mark.gpu

# (coarsest size, periodic, levels): x-pairs of the coarsest level 128, 144,
# 544, 1024, 1088, 2048, 2112 and of thin grids
CASES = [((16, 4, 4), (False,) * 3, 2), ((9, 8, 4), (False, True, False), 3),
         ((33, 8, 4), (False, False, True), 2), ((32, 8, 8), (True, False, False), 2),
         ((34, 8, 8), (False,) * 3, 2), ((64, 8, 8), (True, True, True), 2),
         ((66, 8, 8), (False,) * 3, 2), ((1, 20, 8), (False,) * 3, 2),
         ((2, 16, 12), (True, True, False), 3), ((40, 6, 1), (False,) * 3, 2),
         ((1, 1, 300), (False,) * 3, 2), ((10, 10, 10), (False,) * 3, 3)]


@pytest.mark.parametrize("prec,storage", [("f32", "f32"), ("f32", "bf16"), ("f64", "f64")])
@pytest.mark.parametrize("tail", [4096, 0], ids=["lds", "global"])
@pytest.mark.parametrize("nc,per,nl", CASES, ids=lambda c: str(c).replace(" ", ""))
def test_tail_matches_composed_cycle(nc, per, nl, tail, prec, storage):
    require_gpu()
    n = tuple(v << (nl - 1) for v in nc)
    say(f"tail {n} {per} {prec}/{storage} {tail}")
    L, s, _ = P.random_problem(n, per, seed=sum(n), contrast=2.0, holes=0.1)
    dt = G.GMG_F64 if prec == "f64" else G.GMG_F32
    Ld, sd = dev(rounded(L, prec), prec), dev(rounded(s, prec), prec)
    p = G.gmg_default_params(n, per, dt, l_storage=STORE[storage], anisotropic=0, min_coarse=1,
                             max_levels=nl, tail_cells=tail, coarse_rtol=0.0, nu_coarse=5)
    h = G.gmg_setup(p, Ld)
    levels = G.gmg_num_levels(h)
    assert levels == nl and G.gmg_level_shape(h, nl - 1)[0] == nc
    x = [dev(np.random.default_rng(4).standard_normal(s.shape), prec)]
    xv = x[0].clone()
    sg = [sd]
    for l in range(1, nl):
        m = G.gmg_level_shape(h, l)[0]
        x.append(torch.zeros(m[::-1], dtype=sd.dtype, device=sd.device))
        sg.append(torch.empty_like(x[l]))
    for l in range(nl - 1):
        G.gmg_smooth(h, l, x[l], sg[l], p.nu_pre)
        G.gmg_restrict_residual(h, l, x[l], sg[l], sg[l + 1], x[l + 1])
    G.gmg_smooth(h, nl - 1, x[nl - 1], sg[nl - 1], p.nu_coarse)
    for l in range(nl - 2, -1, -1):
        G.gmg_prolong_correct(h, l, x[l + 1], x[l])
        G.gmg_smooth(h, l, x[l], sg[l], p.nu_post)
    G.gmg_vcycle(h, xv, sd)
    assert torch.equal(xv, x[0])
    h.close()
