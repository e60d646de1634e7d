"""Which launches a set takes follows from its size alone: the planes per work
unit, the z segments and the row tiles a caller or a tuner sets change the
units, not the stages, and never the bits."""
import numpy as np
import pytest

from paper_1711_06203_amd import workloads as W

pytestmark = pytest.mark.gpu

STAGES = ("cons2prim_cfl", "trace_xyz", "trans1_xyz", "riemann_x", "trans2_xyz", "update", "recon_xyz")
DEFAULTS = {"cons2prim_cfl": 2, "trace_xyz": 4, "recon_xyz": 4}


@pytest.fixture(scope="module")
def ctx():
    from paper_1711_06203_amd import ctuppm
    c = ctuppm.Context()
    yield c
    c.close()


def _run(ctx, prob, form):
    """Stages launched by a step, and the state after two."""
    from paper_1711_06203_amd import ctuppm
    s = ctuppm.Solver(ctx, prob, form=form)
    s.step(1)
    ctx.set_timing(True)
    s.step(1)
    ctx.set_timing(False)
    ran = {k for k, (ms, n) in ctx.stage_times().items() if n}
    state = s.state()
    s.close()
    return ran, state


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("n,box,form,small", [
    ((32, 32, 32), (32, 32, 32), "batched", True),    # 136 stage-1 units of one plane
    ((32, 32, 32), (16, 16, 16), "per_box", False),   # several boxes in the per-box form: launches of their own
    ((62, 62, 51), (62, 62, 51), "batched", False),   # 848: just too many, 112 units of eight planes
    ((96, 96, 96), (96, 96, 96), "batched", False),   # 3724, 494 of eight planes
    ((112, 112, 40), (56, 56, 20), "batched", False),
])
def test_stages_do_not_follow_the_tuning(ctx, scheme, n, box, form, small):
    prob = W.kelvin_helmholtz(n=n, box=box, seed=8)
    prob.scheme = scheme
    ran, state = _run(ctx, prob, form)
    assert (("recon_dir" if scheme else "trace_dir") in ran) == small
    try:
        for planes, zseg, ytile in ((8, 1, 0), (64, 1, 0), (2, 3, 5), (1, 1, 1)):
            for st in STAGES:
                ctx.set_stage_planes(st, planes)
            ctx.set_tuning(0, zseg, zseg, ytile)
            got, same = _run(ctx, prob, form)
            assert got == ran, (planes, zseg, ytile)
            assert np.array_equal(same, state), (planes, zseg, ytile)
    finally:
        for st in STAGES:
            ctx.set_stage_planes(st, DEFAULTS.get(st, 1))
        ctx.set_tuning(0, 1, 1)
