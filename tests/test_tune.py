"""What the tuning script stores: a shape that steps the box faster than the library's own choice, and
no other (a stored tile takes the place of the fitted tile and of several steps a launch)."""
import json
import sys

import pytest

from paper_1708_01608_amd import sc, tune


class _FakeSim:
    """Steps in a time that depends on whether a tile was given (seconds a step)."""

    clock = 0.0
    own, tiled = 4e-6, 2e-6

    def __init__(self, tile):
        self.tile = tile

    def seed_nuclei(self, *a):
        pass

    def step(self, n):
        _FakeSim.clock += n * (self.tiled if self.tile else self.own)

    def autotune(self, trials):
        return [dict(tile=(64, 1, 4), variant=1, us=9.0), dict(tile=(128, 1, 1), variant=3, us=3.0)]

    def close(self):
        pass


@pytest.mark.parametrize("own,tiled,stored", [(4e-6, 2e-6, True), (2e-6, 4e-6, False),
                                              (2e-6, 2e-6, False)])
def test_a_shape_is_stored_only_where_it_is_faster(tmp_path, monkeypatch, own, tiled, stored):
    path = tmp_path / "tuned.json"
    keys = [tune.key(9, 128, 128, 1, "f32", c) for c in ("f64", "f32")]
    other = {"q9_64x64x1_f32_f64": {"tile": [64, 1, 4], "variant": 1}}
    path.write_text(json.dumps({keys[0]: {"tile": [64, 1, 1], "variant": 3}, **other}))
    monkeypatch.setattr(tune, "TUNED", str(path))
    monkeypatch.setattr(sc.Sim, "from_spec",
                        classmethod(lambda cls, spec, tile=None, variant=0, **kw: _FakeSim(tile)))
    monkeypatch.setattr(_FakeSim, "own", own)
    monkeypatch.setattr(_FakeSim, "tiled", tiled)
    monkeypatch.setattr(tune.time, "perf_counter", lambda: _FakeSim.clock)
    monkeypatch.setattr(sys, "argv", ["tune", "--workloads", "two_bubble"])
    tune.main()
    table = json.loads(path.read_text())
    assert table.pop("q9_64x64x1_f32_f64") == other["q9_64x64x1_f32_f64"]
    if stored:
        assert sorted(table) == sorted(keys)
        assert all(e["tile"] == [128, 1, 1] and e["variant"] == 3 for e in table.values())
    else:
        assert table == {}
