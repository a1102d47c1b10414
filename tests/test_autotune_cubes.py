"""Host logic of the tile cache's choice of cubes, with the library calls replaced
by recording fakes: entries without the choice are tuned again, cached choices
are made again after the pass's, and a handle that allows no cubes goes without."""
import json

import pytest

from paper_2607_07687_amd import autotune as AT
from paper_2607_07687_amd import gmg as G
from tests.test_autotune_cache import SHAPES, Fake


class CubeFake(Fake):
    def __init__(self, cubes_ok=True):
        super().__init__()
        self.cubes_ok = cubes_ok

    def install(self, monkeypatch):
        super().install(monkeypatch)
        monkeypatch.setattr(G, "gmg_set_cubes", self.set_cubes)

    def autotune(self, h, x, sigma, reps):
        return [dict(r, cube=r["level"] > 0, us_cube=9.0)
                for r in super().autotune(h, x, sigma, reps)]

    def set_cubes(self, h, level, on=True):
        if not self.cubes_ok:
            raise G.GMGError(G.GMG_EINVAL, "no cubes")
        self.calls.append(("cubes", level, on))


def test_entries_without_cube_choice_are_tuned_again(tmp_path, monkeypatch):
    cache = str(tmp_path / "tiles.json")
    old = {f"gfx950|{n[0]}x{n[1]}x{n[2]}|f32|f32":
           dict(ty=8, kchunk=4, us=1.0, pair_kchunk=4, pair_ty=8, us_pair=1.0) for n in SHAPES}
    json.dump(old, open(cache, "w"))
    f = CubeFake()
    f.install(monkeypatch)
    AT.tune(None, None, None, cache=cache)
    assert f.calls == [("autotune", 5)]
    assert [v["cube"] for _, v in sorted(json.load(open(cache)).items())].count(True) == 2


@pytest.mark.parametrize("cubes_ok", [True, False])
def test_cached_cubes_are_set_after_the_pass(cubes_ok, tmp_path, monkeypatch):
    cache = str(tmp_path / "tiles.json")
    CubeFake().install(monkeypatch)
    AT.tune(None, None, None, cache=cache)
    f = CubeFake(cubes_ok)
    f.install(monkeypatch)
    AT.tune(None, None, None, cache=cache)
    assert [c for c in f.calls if c[0] == "cubes"] == (
        [("cubes", 1, True), ("cubes", 2, True)] if cubes_ok else [])
    if cubes_ok:
        order = [c[0] for c in f.calls if c[1] == 1]
        assert order == ["tiles", "pair", "cubes"]
