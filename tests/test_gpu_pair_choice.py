"""GPU checks of how a level's pairs of sweeps are chosen: the default rule, and
what gmg_set_tiles, gmg_set_pair_sweeps and gmg_set_cubes make of it, read back
through gmg_level_cubes; every choice gives bitwise the same sweeps."""
import numpy as np
import pytest

from paper_2607_07687_amd import gmg as G
from paper_2607_07687_amd import problems as P
from tests.gpu_util import dev, require_gpu, rounded, say, torch

pytestmark = pytest.mark.gpu

N, PER = (64, 48, 40), (False, False, False)


def handle(prec, n=N, **kw):
    require_gpu()
    L, s, _ = P.random_problem(n, PER, seed=sum(n), contrast=2.0, holes=0.1)
    dt = G.GMG_F64 if prec == "f64" else G.GMG_F32
    Ld, sd = dev(rounded(L, prec), prec), dev(rounded(s, prec), prec)
    return G.gmg_setup(G.gmg_default_params(n, PER, dt, **kw), Ld), sd


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_calls_choose_the_level_s_sweeps(prec):
    h, sd = handle(prec, tail_cells=0)
    nl = G.gmg_num_levels(h)
    assert nl > 2 and all(G.gmg_level_cubes(h, l) for l in range(nl))
    x0 = dev(np.random.default_rng(3).standard_normal(tuple(sd.shape)), prec)
    want = x0.clone()
    G.gmg_vcycle(h, want, sd)

    def check(level, cubes, what):
        say(f"{prec} level {level} cubes {cubes} after {what}")
        assert G.gmg_level_cubes(h, level) == cubes
        x = x0.clone()
        G.gmg_vcycle(h, x, sd)
        assert torch.equal(x, want)
    # tiles on a level left to the default rule: the sweeps asked for run
    G.gmg_set_tiles(h, 0, 1, 1)
    check(0, False, "gmg_set_tiles")
    G.gmg_set_tiles(h, 1, 4, 2)
    check(1, False, "gmg_set_tiles")
    # kchunk 0: separate sweeps
    G.gmg_set_pair_sweeps(h, 2, 0)
    check(2, False, "gmg_set_pair_sweeps")
    # cubes again; tiles do not undo a choice that was made for pairs
    G.gmg_set_cubes(h, 2, True)
    G.gmg_set_tiles(h, 2, 1, 1)
    check(2, True, "gmg_set_cubes and gmg_set_tiles")
    if prec == "f32":
        G.gmg_set_pair_sweeps(h, 2, 2, 8)
        check(2, False, "gmg_set_pair_sweeps with a pass")
    h.close()


def test_cubes_where_not_allowed():
    h, _ = handle("f32", pair_sweeps=0)
    assert not G.gmg_level_cubes(h, 0)
    for level, on in ((0, True), (99, False), (-1, False)):
        with pytest.raises(G.GMGError) as e:
            G.gmg_set_cubes(h, level, on)
        assert e.value.status == G.GMG_EINVAL
    G.gmg_set_cubes(h, 0, False)
    h.close()
    # large levels take them when told to, with bitwise the same sweeps
    h, sd = handle("f32", (130, 66, 70))
    assert not G.gmg_level_cubes(h, 0)
    xa = torch.zeros_like(sd)
    xb = xa.clone()
    G.gmg_smooth(h, 0, xa, sd, 4)
    G.gmg_set_cubes(h, 0, True)
    G.gmg_smooth(h, 0, xb, sd, 4)
    assert G.gmg_level_cubes(h, 0) and torch.equal(xa, xb)
    h.close()


@pytest.mark.parametrize("prec,n", [("f32", (96, 48, 40)), ("f64", (64, 48, 40)),
                                    ("f32", (65, 33, 24))], ids=str)
def test_autotune_times_cubes_and_round_trips(prec, n, tmp_path):
    # every level that takes cubes by default has them timed, against the best
    # of what else it could run; a handle that is given the cached choices makes
    # the same ones, and then runs the same deferred decisions
    from paper_2607_07687_amd import autotune as AT
    cache = str(tmp_path / "tiles.json")
    h, sd = handle(prec, n, deferred_norm=1, tail_cells=0)
    nl = G.gmg_num_levels(h)
    small = [G.gmg_level_cubes(h, l) for l in range(nl)]
    rep = AT.tune(h, torch.zeros_like(sd), sd, dtype=prec, storage=prec, cache=cache, reps=3)
    for l, r in enumerate(rep):
        say(f"{prec} {n} level {l}: sweep {r['us']:.1f} pass {r['us_pair']:.1f} "
            f"({r['pair_kchunk']}) cubes {r['us_cube']:.1f} ({r['cube']})")
        assert small[l] == (r["us_cube"] > 0)
        if small[l]:
            other = r["us_pair"] if r["pair_kchunk"] else 2 * r["us"]
            assert r["cube"] == (r["us_cube"] < other)
        assert G.gmg_level_cubes(h, l) == r["cube"]
    h2, _ = handle(prec, n, deferred_norm=1, tail_cells=0)
    again = AT.tune(h2, torch.zeros_like(sd), sd, dtype=prec, storage=prec, cache=cache)
    assert all(r["cached"] for r in again)
    assert [G.gmg_level_cubes(h2, l) for l in range(nl)] == [r["cube"] for r in rep]
    xa, xb = torch.zeros_like(sd), torch.zeros_like(sd)
    ra, rb = (G.gmg_solve(a, x, sd, 1e-5, 30) for a, x in ((h, xa), (h2, xb)))
    assert torch.equal(xa, xb) and ra["history"] == rb["history"]
    h.close()
    h2.close()
