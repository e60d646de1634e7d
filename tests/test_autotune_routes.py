"""The per-stage autotuner against a modelled context (no GPU) whose launches
change with a setting: trials that ran other stages are left out."""
import types

import pytest

from paper_1711_06203_amd import autotune

GROUPS = {"trace_xyz": 9, "trace_dir": 9, "update": 0}


class RouteCtx:
    """Above `limit` planes the tracing runs as another stage, and slowly; two
    planes are best otherwise."""

    def __init__(self, limit):
        self.planes = {9: 1, 0: 1}
        self.limit = limit
        self.acc = {}
        self.torch = types.SimpleNamespace(cuda=types.SimpleNamespace(synchronize=lambda: None))

    def stage_planes(self, st):
        return self.planes[GROUPS[st]], GROUPS[st]

    def set_stage_planes(self, st, p):
        self.planes[GROUPS[st]] = int(p)

    def set_timing(self, on):
        if on:
            self.acc = {}

    def step(self, solvers, form, n):
        p = self.planes[9]
        st = "trace_dir" if p > self.limit else "trace_xyz"
        t = 50.0 if p > self.limit else {1: 5.0, 2: 3.0, 4: 4.0, 8: 4.5}[p]
        self.acc = {st: (t * n, n), "update": (1.0 * n, n)}

    def stage_times(self):
        return dict(self.acc)


@pytest.mark.parametrize("limit,best", [(4, 2), (2, 2), (1, 1), (8, 2)])
def test_a_stage_that_did_not_run_is_not_free(limit, best):
    ctx = RouteCtx(limit)
    solver = types.SimpleNamespace(prob=types.SimpleNamespace(boxes=[((0, 0, 0), (95, 95, 95))]))
    out = autotune.tune_stages(ctx, [solver], candidates=(1, 2, 4, 8), steps=1, cache=None)
    assert out["planes"]["trace_xyz"] == best and ctx.planes[9] == best
    assert out["ms_per_step"] == {1: 6.0, 2: 4.0}[best]


def test_no_comparable_trial_keeps_the_setting():
    ctx = RouteCtx(1)
    solver = types.SimpleNamespace(prob=types.SimpleNamespace(boxes=[((0, 0, 0), (95, 95, 95))]))
    out = autotune.tune_stages(ctx, [solver], candidates=(4, 8), steps=1, cache=None)
    assert ctx.planes[9] == 1 and out["planes"]["trace_xyz"] == 1
