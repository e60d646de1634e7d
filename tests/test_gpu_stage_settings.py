"""Settings of the planes per work unit reach the launches that stand for
several stages: each direction of the merged flux launches takes its own
stage's units, the launches of one direction each those of the merged kernels
they replace."""
import itertools

import numpy as np
import pytest

import oracle
from paper_1711_06203_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    from paper_1711_06203_amd import ctuppm
    c = ctuppm.Context()
    yield c
    c.close()


def test_one_setting_by_every_name(ctx):
    planes = lambda st: ctx.stage_planes(st)[0]
    group = lambda st: ctx.stage_planes(st)[1]
    for merged, parts in (("trans2_xyz", ("trans2_x", "trans2_y", "trans2_z")),
                          ("riemann_xyz", ("riemann_x", "riemann_y", "riemann_z"))):
        ctx.set_stage_planes(merged, 5)
        assert [planes(p) for p in parts] == [5, 5, 5]
        ctx.set_stage_planes(parts[0], 3)
        assert planes(merged) == 3 and planes(parts[2]) == 5
        ctx.set_stage_planes(parts[2], 7)
        assert planes(merged) == 3 and planes(parts[0]) == 3
    # a plan that sets z last leaves the others as they are
    assert len({group(st) for st in ("trans2_x", "trans2_y", "trans2_z", "riemann_x", "riemann_z")}) == 5
    for alone, merged in (("trace_dir", "trace_xyz"), ("recon_dir", "recon_xyz"), ("trans1_dir", "trans1_xyz"),
                          ("mol_flux_update", "update")):
        assert group(alone) == group(merged)


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("form", ["batched", "waves"])  # by blocks of one direction, by the merged kernels
def test_each_direction_at_a_depth_of_its_own(ctx, form, scheme):
    prob = W.kelvin_helmholtz(n=(21, 18, 22), box=(12, 18, 11), nspec=1, seed=6)
    prob.scheme = scheme
    ref, _, _ = oracle.run_problem(prob, 2)
    from paper_1711_06203_amd import ctuppm
    for x, y, z in itertools.permutations((1, 4, 64)):
        for st, p in (("riemann_x", x), ("riemann_y", y), ("riemann_z", z), ("trans2_x", x), ("trans2_y", y),
                      ("trans2_z", z)):
            ctx.set_stage_planes(st, p)
        s = ctuppm.Solver(ctx, prob, form=form)
        s.step(2)
        assert np.array_equal(s.state(), ref), (x, y, z)
        s.close()
