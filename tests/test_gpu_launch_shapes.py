"""Every launch of the default mode at other depths of its work units than the
defaults: the blocks of one direction of small sets, the kernels for three
directions above them, the launches with a list per direction, the update that
solves the fluxes.  The stages each case means to cover are checked to have
run; the states are the oracle's, bit for bit."""
import functools

import numpy as np
import pytest

import oracle
from paper_1711_06203_amd import workloads as W

pytestmark = pytest.mark.gpu

SMALL = {0: {"fill_cons2prim_cfl", "trace_dir", "riemann_xyz", "trans1_dir", "trans2_xyz", "update"},
         1: {"fill_cons2prim_cfl", "fill_cons2prim", "recon_dir", "mol_flux_update"},
         2: {"fill_cons2prim_cfl", "fill_cons2prim", "recon_dir", "riemann_xyz", "mol_update"}}
LARGE = {0: {"cons2prim", "trace_xyz", "species_xyz", "riemann_xyz", "trans1_xyz", "trans2_xyz", "update"},
         1: {"cons2prim", "recon_xyz", "mol_flux_update"},
         2: {"cons2prim", "recon_xyz", "species_xyz", "riemann_xyz", "mol_update"}}
GROUPS = ("trace_xyz", "trans1_xyz", "riemann_xyz", "trans2_xyz", "update", "cons2prim")


def _problem(case, n, box):
    # 0: CTU with species (two-shock), 1: method of lines, 2: with species
    prob = W.kelvin_helmholtz(n=n, box=box, seed=9, nspec=(2, 0, 1)[case])
    prob.scheme, prob.riemann = (0, 1, 2)[case], (1, 0, 1)[case]
    return prob


@functools.lru_cache(maxsize=None)
def _reference(case, n, box, steps):
    ref, _, _ = oracle.run_problem(_problem(case, n, box), steps)
    return ref


def _run(prob, form, setting, steps):
    from paper_1711_06203_amd import ctuppm
    ctx = ctuppm.Context()
    try:
        for st, p in setting.items():
            ctx.set_stage_planes(st, p)
        s = ctuppm.Solver(ctx, prob, form=form)
        ctx.set_timing(True)
        s.step(steps)
        ctx.set_timing(False)
        ran = {k for k, (ms, m) in ctx.stage_times().items() if m}
        out = [s.state()] + (s.state_patches() if prob.fine_boxes else [])
        s.close()
    finally:
        ctx.close()
    return out, ran


SETTINGS = [{g: p} for g in GROUPS for p in (2, 5)] + [dict.fromkeys(GROUPS, p) for p in (1, 64)] + [
    {"trace_xyz": 8, "trans1_xyz": 3, "riemann_y": 5, "riemann_z": 2, "trans2_x": 4, "trans2_z": 7, "update": 6}]


@pytest.mark.parametrize("setting", SETTINGS, ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items()))
@pytest.mark.parametrize("case", [0, 1, 2])
def test_small_sets_and_waves(case, setting):
    n, box = (30, 27, 22), (15, 14, 22)
    ref = _reference(case, n, box, 2)
    for form, stages in (("batched", SMALL[case]), ("waves", LARGE[case])):
        got, ran = _run(_problem(case, n, box), form, setting, 2)
        assert stages <= ran, form
        assert np.array_equal(got[0], ref), form


@pytest.mark.parametrize("setting", [{"trans2_xyz": 2, "trace_xyz": 2}, dict.fromkeys(GROUPS, 8)],
                         ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items()))
@pytest.mark.parametrize("case", [0, 1, 2])
def test_batched_sets_above_the_small_ones(case, setting):
    n, box = (62, 62, 51), (62, 62, 51)
    got, ran = _run(_problem(case, n, box), "batched", setting, 1)
    assert LARGE[case] - {"cons2prim"} <= ran
    assert np.array_equal(got[0], _reference(case, n, box, 1))


@pytest.mark.parametrize("setting", [{"trans2_xyz": 3}, {"trace_xyz": 6, "riemann_xyz": 2}, dict.fromkeys(GROUPS, 64)],
                         ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items()))
def test_two_levels(setting):
    prob = W.cloud_wind(n=32, box=16, fine_box=8, fine_region=((10, 10, 10), (22, 22, 22)), nspec=1)
    got, ran = _run(prob, "batched", setting, 2)
    assert LARGE[0] <= ran
    rc, rf, _, _ = oracle.run_two_level(prob, 2)
    assert np.array_equal(got[0], rc) and np.array_equal(got[1], rf)
