"""The launch tuner tries the library's own chunk rule (tile 0), alone and on its other grids, and
keeps it where it is the fastest: any tile above 0 is taken literally, so that few leptons would
share few wavefronts.  Scripted step times; no GPU."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_1412_6426_amd import autotune as AT


class FakeEngine:
    stream = 0

    def __init__(self, best):
        self.best, self.shape = best, None

    def counts(self):
        return np.array([[1 << 17, 0, 0]], dtype=np.int64)

    def set_arena(self, divisor):
        pass

    def step(self, field, params):
        self.shape = (params.tile, params.grid_blocks)

    def stats(self):
        return {"advanced": [1 << 17, 0, 0], "dropped": 0}


@pytest.mark.parametrize("grid", [0, 512, 2048])
def test_the_rule_is_tried_and_kept(grid):
    cands = AT.default_candidates(256)
    assert cands[0] == AT.DEFAULT_SHAPE and (0, grid, 0, 0) in cands
    assert len(set(cands)) == len(cands)
    e = FakeEngine((0, grid))
    timer = SimpleNamespace(start=lambda s: None,
                            stop_ms=lambda s: 1.0 if e.shape == e.best else 2.0)
    params = SimpleNamespace(tile=0, grid_blocks=0, refill_min=0)
    sched = AT.tune_run(e, None, params, 60, cands, timer=timer, sync=lambda: None)
    assert [s[:2] for s in sched.choices.values()] == [(0, grid)]
