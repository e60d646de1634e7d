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


class MergedCtx:
    """Launches that stand for several stages: each part has its own best depth."""
    GROUPS = {"riemann_x": 2, "riemann_y": 2, "riemann_z": 5, "riemann_xyz": 2, "trans1_xyz": 2, "trans1_dir": 2,
              "trans2_x": 6, "trans2_y": 7, "trans2_z": 8, "trans2_xyz": 6, "trace_xyz": 9, "trace_dir": 9, "update": 0}
    LAUNCHES = {"riemann_xyz": (2, 5), "trans1_dir": (2,), "trans2_xyz": (6, 7, 8), "trace_dir": (9,), "update": (0,)}
    BEST = {2: 1, 5: 1, 6: 4, 7: 4, 8: 4, 9: 2, 0: 1}

    def __init__(self):
        self.planes = {g: 2 for g in set(self.GROUPS.values())}
        self.planes[9] = 4
        self.set_by_caller = set()
        self.acc = {}
        self.torch = types.SimpleNamespace(cuda=types.SimpleNamespace(synchronize=lambda: None))

    def stage_planes(self, st):
        return self.planes[self.GROUPS[st]], self.GROUPS[st]

    def set_stage_planes(self, st, p):
        for g in {"riemann_xyz": (2, 5), "trans2_xyz": (6, 7, 8)}.get(st, (self.GROUPS[st],)):
            self.planes[g] = int(p)
            self.set_by_caller.add(g)

    def set_timing(self, on):
        if on:
            self.acc = {}

    def step(self, solvers, form, n):
        for st, gs in self.LAUNCHES.items():
            self.acc[st] = (n * sum(1.0 + abs(self.planes[g] - self.BEST[g]) for g in gs), n)

    def stage_times(self):
        return dict(self.acc)


def test_settings_of_merged_launches_are_tuned_and_cached_alike(tmp_path):
    solver = types.SimpleNamespace(prob=types.SimpleNamespace(boxes=[((0, 0, 0), (47, 47, 47))]))
    fresh, cached = MergedCtx(), MergedCtx()
    cache = str(tmp_path / "tuning.json")
    out = autotune.tune_stages(fresh, [solver], candidates=(1, 2, 4), steps=1, cache=cache)
    assert fresh.planes == MergedCtx.BEST
    # every setting reported was timed, and holds what it says
    assert set(out["planes"]) == {"riemann_x", "riemann_y", "riemann_z", "trans1_xyz", "trans2_x", "trans2_y",
                                  "trans2_z", "trace_xyz", "update"}
    assert all(fresh.stage_planes(st)[0] == p for st, p in out["planes"].items())
    again = autotune.tune_stages(cached, [solver], steps=1, cache=cache)
    assert again["cached"] and again["planes"] == out["planes"]
    assert cached.planes == fresh.planes and cached.set_by_caller == fresh.set_by_caller


def test_no_setting_of_a_stage_that_never_ran(tmp_path):
    """The method of lines takes its fluxes in the update: riemann_x stays as it was."""
    ctx = MergedCtx()
    ctx.GROUPS = dict(ctx.GROUPS, mol_flux_update=0, mol_update=0, recon_dir=9, recon_xyz=9)
    ctx.LAUNCHES = {"recon_dir": (9,), "mol_flux_update": (0,)}
    solver = types.SimpleNamespace(prob=types.SimpleNamespace(boxes=[((0, 0, 0), (47, 47, 47))]))
    out = autotune.tune_stages(ctx, [solver], candidates=(1, 2, 4), steps=1, cache=str(tmp_path / "t.json"))
    assert out["planes"] == {"recon_xyz": 2, "mol_update": 1} and ctx.set_by_caller == {0, 9}


class AdaptiveCtx(RouteCtx):
    """A small set: the tracing runs at one plane, its best, until it is set; its
    default reads 4.  A tuned step is a little slower than the start."""

    def __init__(self):
        super().__init__(limit=8)
        self.planes[9] = 4
        self.is_set = False

    def set_stage_planes(self, st, p):
        super().set_stage_planes(st, p)
        self.is_set = True

    def step(self, solvers, form, n):
        p = self.planes[9] if self.is_set else 1
        self.acc = {"trace_xyz": ({1: 5.0, 2: 6.0, 4: 8.0, 8: 9.0}[p] * n, n),
                    "update": ((1.1 if self.is_set else 1.0) * n, n)}


def test_the_starting_setting_is_kept_only_if_setting_it_is_no_slower():
    ctx = AdaptiveCtx()
    solver = types.SimpleNamespace(prob=types.SimpleNamespace(boxes=[((0, 0, 0), (47, 47, 47))]))
    out = autotune.tune_stages(ctx, [solver], candidates=(1, 2, 4, 8), steps=1, cache=None)
    assert out["planes"]["trace_xyz"] == 1 and ctx.planes[9] == 1
    assert out["start_ms_per_step"] == 6.0 and out["ms_per_step"] == 6.1
