"""The autotuner times each of the face-flux pass' block shapes once, not the
many tiles that name the same kernel, and keeps the default, which lets the grid
or the batch decide, unless a shape is clearly faster."""

import pytest

from paper_2110_10191_amd import tune


class State:
    def clone(self):
        return self

    def copy_(self, other):
        return self


class FakeSim:
    ctx = None

    def __init__(self):
        self.tiles = dict(tune.DEFAULT)
        self.set = []

    def get_dt(self, P):
        return 1.0

    def step(self, P, dt, want_dt_next=True):
        return dt

    def set_tiles(self, cls, tx, ty):
        self.tiles[cls] = (tx, ty)
        self.set.append((cls, (tx, ty)))


@pytest.mark.parametrize("narrow_ms,want", [(0.985, (64, 8)), (0.9, (16, 8))], ids=["within_the_margin", "clearly_faster"])
def test_each_shape_is_timed_and_the_default_kept_on_ties(monkeypatch, narrow_ms, want):
    cost = {(64, 8): 1.0, (128, 4): 1.4, (32, 8): 0.995, (16, 8): narrow_ms}
    monkeypatch.setattr(tune, "time_classes", lambda sim, P, dt, classes, steps, repeats:
                        [cost[sim.tiles["sweep"]] if classes == tune.SWEEP_CLASSES else 2.0])
    sim = FakeSim()
    tiles, timings = tune.tune_sim(sim, State(), repeats=2)
    assert tiles == {"sweep": want, "update": tune.DEFAULT["update"]}
    assert timings["sweep"] == cost[want]
    swept = {t for cls, t in sim.set if cls == "sweep"}
    assert swept == set(tune.SWEEP_SHAPES) == set(cost)
    assert swept <= set(tune.candidates("sweep")) and tune.SWEEP_SHAPES[0] == tune.DEFAULT["sweep"]
    assert sim.tiles["sweep"] == want


def test_search_over_given_sweep_tiles():
    calls = []

    def measure(t):
        calls.append(t["sweep"])
        return 1.0 - 0.01 * (t["sweep"] == (32, 8))

    tiles, _ = tune.search(measure, repeats=1, sweep=tune.SWEEP_SHAPES, margin=tune.SWEEP_MARGIN)
    assert tiles["sweep"] == tune.DEFAULT["sweep"] and set(calls) == set(tune.SWEEP_SHAPES)
