"""The tuner's choices against timings given for every candidate (host): the
open batch is found where it is the fastest, and lengths chosen on a probe
batch mean the same planes in any other.
"""
from types import SimpleNamespace

import pytest

import paper_2006_02602_amd as C
from paper_2006_02602_amd import autotune


class Fake:
    """A batch whose time a step is cost(shapes, nblocks); points where every member is open."""

    def __init__(self, grids, cost, points=5):
        self.grids, self.cost, self.points, self.tried = grids, cost, points, []
        self.retile([(0, 0)] * len(grids))

    def retile(self, shapes):
        self.shapes = [(int(kc), int(ti)) for kc, ti in shapes]
        self.tried.append(self.shapes)
        self.handle = SimpleNamespace(points=self.points if all(s == (0, 0) for s in self.shapes) else 0)

    def step(self, steps, nblocks=0):
        self.ms = self.cost(self.shapes, nblocks)


@pytest.fixture
def clock(monkeypatch):
    now = {}

    def _time(fn, reps):
        fn()
        return now["batch"].ms
    monkeypatch.setattr(autotune, "_time", _time)
    return now


@pytest.mark.parametrize("points,open_ms,open_wins", [(5, 1.0, True), (5, 9.0, False), (0, 1.0, False)])
def test_tuned_batch_is_no_slower_than_the_open_one(clock, tmp_path, points, open_ms, open_wins):
    dtype, keys = C.CAV_F64, ["a", "b", "a"]
    wide = autotune.ti_candidates(dtype)[0]

    def cost(shapes, nb):
        if all(s == (0, 0) for s in shapes):
            return open_ms + (0.0 if nb == 512 else 0.5)
        return 2.0 + sum(abs(kc - 8) + (ti != wide) for kc, ti in shapes) + (0.0 if nb == 256 else 0.25)

    def batch():
        return Fake([C.Grid(40, 30, 20), C.Grid(9, 9, 33), C.Grid(40, 30, 20)], cost, points)
    path = str(tmp_path / "cache.json")
    for _ in range(2):                                    # tuned, then from the cache
        b = clock["batch"] = batch()
        shape, nb, _ = autotune.tune_batch(b, keys, dtype, cache_path=path)
        want = ({"a": (0, 0), "b": (0, 0)}, 512) if open_wins else ({"a": (wide, 8), "b": (wide, 8)}, 256)
        assert (shape, nb) == want
        assert b.shapes == [(shape[k][1], shape[k][0]) for k in keys]      # left with the chosen work list


@pytest.mark.parametrize("edge", [2, 3, 24, 32, 50])
def test_lengths_of_a_probe_batch_hold_in_any_batch(clock, monkeypatch, edge):
    tried = []

    class Probe:
        def __init__(self, members):
            (_, _, self.kc, self.ti) = members[0]
            tried.append((self.ti, self.kc))
            clock["batch"] = self

        def init(self, seeds):
            return self

        def step(self, steps):
            self.ms = 100.0 - self.kc                     # the longest is the fastest
    monkeypatch.setattr(autotune, "Batch", Probe)
    out = autotune.tune_shapes([edge], C.CAV_F32)
    assert all(0 < kc <= edge for _, kc in tried)
    assert out[edge][1] == edge
    assert len(tried) == len(set(tried))
