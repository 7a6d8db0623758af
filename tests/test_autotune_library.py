"""The tuners against the library's own choice (every schedule field 0), which runs small
meshes in the tile kernels whatever the number of passes: host logic, with the times
made up."""
import types

import pytest

from paper_1208_2407_amd import autotune


class FakePlan:
    def __init__(self, order=2, n=256):
        self.problem = types.SimpleNamespace(nx=n, ny=n, nz=1, order=order, bc=0)
        self.dtype = "c64"
        self.fields = None

    def set_schedule(self, *fields):
        self.fields = fields

    def passes(self, steps):  # the same count on every route, as at fourth order
        return steps, False

    def schedule(self):
        return autotune.LIBRARY_REPORTS if self.fields == (0, 0, 0, 0) else self.fields


class FakeState:
    device = None

    def clone(self):
        return self


@pytest.fixture
def tuner(monkeypatch, tmp_path):
    import torch
    monkeypatch.setenv("TSQ_AUTOTUNE_CACHE", str(tmp_path / "cache.json"))
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda device: types.SimpleNamespace(gcnArchName="gfx950:none"))
    times = {}

    def time(plan, *args, **kw):
        schedule = args[-1] if len(args) == 3 and isinstance(args[-1], tuple) else args[1]
        return times.get(tuple(schedule), 1.0 + 0.01 * schedule[0])

    monkeypatch.setattr(autotune, "time_schedule", time)
    monkeypatch.setattr(autotune, "time_schedule_td", time)
    return times


@pytest.mark.parametrize("order", [2, 4])
def test_tune_keeps_faster_tile_kernels(tuner, order):
    tuner[(0, 0, 0, 0)] = 0.5
    plan = FakePlan(order)
    for _ in range(2):  # timed, then from the cache
        assert autotune.tune(plan, FakeState())[0] == (0, 0, 0, 0)
        assert plan.fields == (0, 0, 0, 0)
        plan.fields = None


@pytest.mark.parametrize("library", [0.99, 1.06, 3.0])
def test_tune_keeps_schedules_the_library_does_not_beat(tuner, library):
    tuner[(0, 0, 0, 0)] = library
    plan = FakePlan()
    tuner[(1, 64, 1, 1)] = 0.9  # a segment height of the shallowest schedule
    assert autotune.tune(plan, FakeState())[0] == (1, 64, 1, 1) == plan.fields


def test_tune_td_leaves_the_default_schedule_to_the_library(tuner):
    tuner[(0, 0, 0, 0)] = 0.5
    plan = FakePlan()
    for _ in range(2):
        sched, table = autotune.tune_td(plan, FakeState(), [0.1] * 8)
        assert sched in autotune.TD_CANDIDATES and sched == plan.schedule()
        assert plan.fields == (0, 0, 0, 0) and len(table) == len(autotune.TD_CANDIDATES)
        plan.fields = None
    # candidates of the caller are taken as they are
    assert autotune.tune_td(plan, FakeState(), [0.1] * 8, candidates=[(5, 0, 1, 1)], use_cache=False)[0] == plan.fields
    tuner[(3, 0, 1, 2)] = 0.1
    assert autotune.tune_td(plan, FakeState(), [0.1] * 8, use_cache=False)[0] == (3, 0, 1, 2) == plan.fields
