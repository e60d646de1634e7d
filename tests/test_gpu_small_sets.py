"""Small sets take dt and the commit in the last blocks of the conversion and
the update, and their ghost fill, through the boundaries too, in the
conversion's launch.
Each value takes the same operations as in the launches of their own that
larger sets use, so states, ghost cells, dt and counters are compared bit for
bit, with the oracle and with the split stages."""
import numpy as np
import pytest

import oracle
from paper_1711_06203_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1711_06203_amd import ctuppm
    c = ctuppm.Context()
    yield c
    c.set_fused(1)
    c.close()


def _step(ctx, prob, form, fused, steps):
    from paper_1711_06203_amd import ctuppm
    ctx.set_fused(fused)
    s = ctuppm.Solver(ctx, prob, form=form)
    s.step(steps)
    out = [s.state(), s.counters(), np.array([s.dt()]), s.UA.cpu().numpy()]  # with the ghost cells of U^n
    s.close()
    return out


@pytest.mark.parametrize("form", ["per_box", "batched", "graph"])
@pytest.mark.parametrize("scheme", [0, 1, 2])
@pytest.mark.parametrize("n,box", [
    ((4, 4, 4), (4, 4, 4)),          # the smallest periodic extent: every ghost cell its own box's
    ((15, 4, 5), (15, 4, 5)),        # fewer update units than counters
    ((16, 16, 16), (16, 16, 16)),    # sixteen units, one a counter
    ((17, 15, 16), (17, 15, 16)),
    ((20, 9, 14), (7, 9, 5)),        # ghost cells from several boxes
])
def test_dt_commit_and_ghosts(ctx, form, scheme, n, box):
    prob = W.kelvin_helmholtz(n=n, box=box, seed=7, nspec=scheme)
    prob.scheme = scheme
    got = _step(ctx, prob, form, 1, 3)
    split = _step(ctx, prob, form, 0, 3)
    ref, dts, _ = oracle.run_problem(prob, 3)
    assert np.array_equal(got[0], ref) and got[2][0] == dts[-1]
    for a, b in zip(got, split):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("form", ["per_box", "batched", "graph"])
@pytest.mark.parametrize("scheme", [0, 1])
def test_rejected_step_is_not_committed(ctx, form, scheme):
    from paper_1711_06203_amd import ctuppm
    ctx.set_fused(1)
    prob = W.serving_request(seed=4, n=11)
    prob.scheme = scheme
    s = ctuppm.Solver(ctx, prob, form=form)
    s.set_fail_hook(1)
    s.step_guarded(1)
    with pytest.raises(ctuppm.Rejected):
        for _ in range(50):
            s.step_guarded(1)
            ctx.torch.cuda.synchronize()
    assert s.rejections() == 1
    s.step_guarded(1)  # the hook fired once: the step is redone
    assert s.counters()[5] == 2
    ref, _, _ = oracle.run_problem(prob, 2)
    assert np.array_equal(s.state(), ref)
    s.close()


def test_many_small_problems_in_one_set(ctx):
    from paper_1711_06203_amd import ctuppm
    ctx.set_fused(1)
    probs = [W.serving_request(seed=s, n=4 + s % 9) for s in range(21)]  # two launches of segments
    solvers = [ctuppm.Solver(ctx, p, form="batched") for p in probs]
    for _ in range(3):
        ctx.step(solvers, "batched", 1, guarded=True)
    for s, p in zip(solvers, probs):
        ref, dts, _ = oracle.run_problem(p, 3)
        assert np.array_equal(s.state(), ref) and s.dt() == dts[-1]
        s.close()


@pytest.mark.parametrize("n,box", [
    ((62, 62, 49), (62, 62, 49)),   # 816 units of 256 cells with a halo of one: blocks of one direction
    ((62, 62, 50), (62, 62, 50)),   # 832: the last set that takes them
    ((62, 62, 51), (62, 62, 51)),   # 848: one kernel for the three directions
    ((13, 4, 5), (13, 4, 5)),       # one part of a block a plane (a mirror image needs four cells of domain)
    ((14, 14, 9), (5, 14, 2)),
])
@pytest.mark.parametrize("scheme,riemann,limiter,steepen,nspec", [
    (0, 0, 0, 0, 2), (0, 1, 1, 0, 0), (0, 0, 0, 1, 0), (1, 0, 1, 0, 1), (2, 1, 0, 0, 0),
])
def test_blocks_of_one_direction(ctx, n, box, scheme, riemann, limiter, steepen, nspec):
    prob = W.kelvin_helmholtz(n=n, box=box, seed=11, nspec=nspec)
    prob.scheme, prob.riemann, prob.limiter, prob.steepen = scheme, riemann, limiter, steepen
    prob.bc_lo, prob.bc_hi = (W.BC_OUTFLOW, W.BC_REFLECT, W.BC_REFLECT), (W.BC_REFLECT, W.BC_OUTFLOW, W.BC_REFLECT)
    got = _step(ctx, prob, "batched", 1, 2)
    split = _step(ctx, prob, "batched", 0, 2)
    for a, b in zip(got, split):
        assert np.array_equal(a, b, equal_nan=True)
    if prob.zones < 10000:
        ref, dts, _ = oracle.run_problem(prob, 2)
        assert np.array_equal(got[0], ref) and got[2][0] == dts[-1]


P, O, R, I = W.BC_PERIODIC, W.BC_OUTFLOW, W.BC_REFLECT, W.BC_INFLOW


@pytest.mark.parametrize("form", ["per_box", "batched", "graph"])
@pytest.mark.parametrize("n,box", [
    ((12, 10, 9), (12, 10, 9)),      # one box: every ghost cell an image of its own
    ((12, 10, 9), (5, 4, 9)),        # images that lie in other boxes
    ((12, 10, 9), (1, 3, 2)),        # boxes thinner than the ghost layers, some beside the walls
    ((4, 5, 4), (3, 5, 2)),          # the smallest domain a mirror image fits
])
@pytest.mark.parametrize("bc_lo,bc_hi", [
    ((O, O, O), (O, O, O)), ((R, R, R), (R, R, R)), ((I, I, I), (I, I, I)),
    ((O, P, P), (O, P, P)), ((P, P, R), (P, P, R)),
    ((R, I, O), (I, O, R)), ((I, R, P), (R, O, P)), ((O, R, I), (I, I, R)), ((R, P, I), (O, P, R)),
])
def test_ghost_cells_through_boundaries(ctx, form, n, box, bc_lo, bc_hi):
    """Edge and corner ghost cells too: U^n with its ghost cells is compared."""
    scheme = sum(bc_lo) % 3
    prob = W.kelvin_helmholtz(n=n, box=box, seed=n[0] + box[0], nspec=2)
    prob.scheme, prob.bc_lo, prob.bc_hi = scheme, bc_lo, bc_hi
    prob.inflow, prob.inflow_X = (1.25, 0.5, -0.25, 0.125, 2.0), (0.25, 0.75)
    got = _step(ctx, prob, form, 1, 2)
    split = _step(ctx, prob, form, 0, 2)
    ref, dts, _ = oracle.run_problem(prob, 2)
    assert np.array_equal(got[0], ref) and got[2][0] == dts[-1]
    for a, b in zip(got, split):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("n,box,nspec", [
    ((101, 101, 93), (101, 101, 93), 0),    # 3720 update units, 1.2 M cells with ghosts: one launch
    ((96, 96, 114), (96, 96, 114), 0),      # 4104 units: launches of their own
    ((84, 72, 64), (16, 16, 16), 1),        # 1.42 M cells with ghosts in boxes of 16^3 and less
    ((90, 80, 64), (16, 16, 16), 0),        # 1.59 M
    ((96, 80, 64), (16, 16, 16), 0),        # 1.66 M: too many
])
def test_ghosts_with_conversion_at_the_edges_of_the_rule(ctx, n, box, nspec):
    prob = W.kelvin_helmholtz(n=n, box=box, seed=5, nspec=nspec)
    prob.bc_lo, prob.bc_hi = (O, P, R), (R, P, O)
    got = _step(ctx, prob, "batched", 1, 1)
    split = _step(ctx, prob, "batched", 0, 1)
    for a, b in zip(got, split):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("bc", [O, R, I])
def test_bare_parts_of_the_domain_keep_the_callers_ghosts(ctx, bc):
    """Ghost cells over a part of the domain without boxes have no source: they
    stay what the caller made them, and the set keeps its launches."""
    from paper_1711_06203_amd import ctuppm
    prob = W.kelvin_helmholtz(n=(18, 16, 12), box=(9, 8, 6), seed=2)
    prob.boxes = prob.boxes[:-1]
    prob.bc_lo, prob.bc_hi = (bc, O, P), (O, bc, P)
    out = []
    for fused in (1, 0):
        ctx.set_fused(fused)
        s = ctuppm.Solver(ctx, prob, form="batched")
        s.UA[ctx.torch.isnan(s.UA) | (s.UA == 0.0)] = 0.125
        s.step(2)
        out.append((s.UA.cpu().numpy(), s.UB.cpu().numpy(), s.counters(), s.dt()))
        s.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b, equal_nan=True)
