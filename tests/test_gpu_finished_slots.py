"""GPU check that a recorded cycle slot whose solve has finished is cheap: the
inner cycles of a refinement step beyond the last needed one, which every kernel
leaves at once, cost no more with the levels' sweeps in pairs on cubes than as
twice as many separate launches."""
import pytest

from paper_2607_07687_amd import gmg as G
from paper_2607_07687_amd import problems as P
from tests.gpu_util import dev, require_gpu, say, torch

pytestmark = pytest.mark.gpu


def slot_us(L, s, n, per, **kw):
    """Time of one finished slot: 64 against 8 recorded inner cycles."""
    sd, ms = dev(s, "f64"), {}
    x = torch.zeros_like(sd)
    h = G.gmg_setup(G.gmg_default_params(n, per, G.GMG_F64, cycle_dtype=G.GMG_F32, **kw),
                    dev(L, "f64"))
    for slots in (8, 64):
        best = float("inf")
        for rep in range(6):  # the first records the graph
            x.zero_()
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in "ab")
            e0.record()
            info = G.gmg_solve_ir(h, x, sd, 1e-10, 20, slots, 1e-4)
            e1.record()
            e1.synchronize()
            assert info["status"] == "GMG_OK" and max(info["inner_cycles"]) <= 8
            if rep:
                best = min(best, e0.elapsed_time(e1))
        ms[slots] = best
    h.close()
    return 1e3 * (ms[64] - ms[8]) / (56 * info["outer"]), info["outer"]


def test_finished_slots_cost_no_more_with_cubes():
    require_gpu()
    n = (256, 64, 64)
    L, s, per = P.sphere_box(n, (128.0, 32.0, 32.0), 10.0, "uniform", 3)
    cubes, outer = slot_us(L, s, n, per)
    single, _ = slot_us(L, s, n, per, pair_sweeps=0)
    say(f"finished slot: {cubes:.1f} us with pairs on cubes, {single:.1f} us as separate sweeps "
        f"({outer} refinement steps)")
    assert cubes <= single
