"""The tuner keeps the default shapes unless another candidate is at least 2%
faster, and the committed table holds to that."""
import io

import pytest

from paper_1405_0194_amd import lattice, tune


@pytest.mark.parametrize("gain,chosen", [(0.0, False), (0.0001, False), (0.0199, False), (0.0201, True), (0.3, True)])
def test_margin(monkeypatch, gain, chosen):
    fast = dict(leaf_cols=64, panel_width=64, tile_rows=64)
    monkeypatch.setattr(tune, "time_candidate", lambda s, P, o, reps=3, device="cuda": (
        0.01 if o == fast else 0.01 * (1 + gain) if o == tune.DEFAULTS else 0.02, None))
    s = lattice.make_system("honeycomb", (3, 3), 5, 3.0, 5)
    cache = {}
    key, ent = tune.tune_system(s, 40, cache, log=io.StringIO())
    assert ent is cache[key] and ent["options"] == (fast if chosen else tune.DEFAULTS)
    assert ent["seconds"] == (0.01 if chosen else ent["default_seconds"])


def test_candidates_without_the_defaults(monkeypatch):
    monkeypatch.setattr(tune, "time_candidate", lambda s, P, o, reps=3, device="cuda": (1.0 / o["leaf_cols"], None))
    s = lattice.make_system("honeycomb", (3, 3), 5, 3.0, 5)
    only = dict(leaf_cols=(64, 256), panel_width=(32,), tile_rows=(64,))
    key, ent = tune.tune_system(s, 40, {}, candidates=only, log=io.StringIO())
    assert ent["options"]["leaf_cols"] == 256 and ent["default_seconds"] is None


def test_committed_table():
    cache = tune.load_cache()
    assert len(cache) >= 28
    for key, ent in cache.items():
        times = {tuple(sorted(t["options"].items())): t["seconds"] for t in ent["trials"]}
        assert ent["seconds"] == times[tuple(sorted(ent["options"].items()))], key
        if ent["options"] != tune.DEFAULTS:
            assert ent["default_seconds"] >= 1.02 * ent["seconds"], key
        else:
            assert ent["seconds"] <= 1.02 * min(times.values()), key
