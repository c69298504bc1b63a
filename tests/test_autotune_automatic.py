"""The tile autotuner beside the library's own choice: it is timed for every
mesh of the library, batched or not, returned where it is the fastest, and is
what the cache calls the default; entries written for other kernels, or without
that candidate, are not read."""
import json

import pytest

from paper_1204_5125_amd import autotune, glnk


class Info:
    def __init__(self, *a, **k):
        pass

    def info(self):
        return {"nlev": 3, "sizes": [4225, 700, 90], "nnz": [0, 0, 0], "ncolors": [2, 4, 5]}


@pytest.fixture
def mesh(monkeypatch):
    m = glnk.Mesh.__new__(glnk.Mesh)
    m._h, m.dim, m.shape, m.n = None, 2, (65, 65), 4225
    monkeypatch.setattr(glnk, "Precond", Info)
    monkeypatch.setattr(autotune, "_key", lambda mesh, p, mc: "dev")
    return m


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("auto_time", [0.1, 0.9])
def test_automatic_choice_is_a_candidate(mesh, monkeypatch, tmp_path, batch, auto_time):
    calls = []

    def fake(mesh, psi, pre, tiles, iters=24, reps=3):
        calls.append(tuple(tiles))
        return auto_time if tuple(tiles) == autotune.AUTO else 0.5 + 0.01 * len(calls)

    monkeypatch.setattr(autotune, "time_tiles", fake)
    cache = tmp_path / "t.json"
    # what earlier kernels left under their key
    cache.write_text(json.dumps({"dev" + ("|batch" if batch else ""): {"tiles": [1, 64, 0, 0]}}))
    best = autotune.tune(mesh, None, cache=str(cache), batch=batch)
    assert calls.count(autotune.AUTO) == 1 and len(calls) > 1
    assert (best == autotune.AUTO) == (auto_time < 0.5)
    new = [v for v in json.loads(cache.read_text()).values() if "us_per_iteration" in v]
    assert len(new) == 1 and tuple(new[0]["tiles"]) == best
    assert new[0]["default_us_per_iteration"] == pytest.approx(auto_time * 1e6)
    calls.clear()
    assert autotune.tune(mesh, None, cache=str(cache), batch=batch) == best and calls == []
    # without it, and not from that entry
    assert autotune.tune(mesh, None, cache=str(cache), batch=batch, auto=False) != autotune.AUTO
    assert autotune.AUTO not in calls and calls
