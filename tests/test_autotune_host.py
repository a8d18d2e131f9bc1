"""The batch autotuner without a GPU: what it sweeps, and caches with and without entries it no longer needs."""
import json

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as W  # noqa: E402
from paper_2504_12013_amd import autotune, jet  # noqa: E402


class Batch:
    """Records options and refinements."""

    def __init__(self):
        self.options, self.refined = {}, []

    def set_option(self, option, value):
        self.options[option] = value

    def refine(self, parts, replays=8, **kw):
        self.refined.append((replays, tuple(sorted(self.options.items()))))


@pytest.fixture
def batch(monkeypatch):
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    return Batch()


HGS = [W.random_hypergraph(200, 300, 4, 1), W.random_hypergraph(300, 400, 8, 2)]
PARTS = [torch.from_numpy(np.zeros(h.n, np.int32)) for h in HGS]


def test_only_knobs_that_change_the_time_are_swept(batch, tmp_path):
    path = str(tmp_path / "c.json")
    key, settings = autotune.tuned(batch, HGS, PARTS, cache_path=path)
    timed = {o for _, o in batch.refined}
    assert len(batch.refined) == 2 * len(timed)  # every setting once, after a warm-up: nothing else varies
    assert {r for r, _ in batch.refined} == {8}
    assert set(settings) == set(autotune.KNOBS) | {"replays"}
    assert "replays" not in autotune.KNOBS
    again = Batch()
    assert autotune.tuned(again, HGS, PARTS, cache_path=path) == (key, settings) and not again.refined


@pytest.mark.parametrize("extra", [{}, {"replays": 32}])
def test_older_caches_are_read(batch, tmp_path, extra):
    path = tmp_path / "c.json"
    entry = {"grid": 4096, "lane_degree": 0, "apply_divisor": 16, "rb_slots": 2, "seconds": {}}
    path.write_text(json.dumps({autotune.shape_key(HGS): dict(entry, **extra)}))
    _, settings = autotune.tuned(batch, HGS, PARTS, cache_path=str(path))
    assert not batch.refined
    assert {k: settings[k] for k in autotune.KNOBS} == {k: entry[k] for k in autotune.KNOBS}
    assert batch.options == {jet.JET_OPT_GRID: 4096, jet.JET_OPT_CAND_LANE_DEGREE: 0, jet.JET_OPT_APPLY_DIVISOR: 16,
                             jet.JET_OPT_RB_SLOTS: 2}


def test_stored_choices_are_complete():
    with open(autotune.DEFAULT_CACHE) as f:
        for entry in json.load(f).values():
            assert set(autotune.KNOBS) <= set(entry)
