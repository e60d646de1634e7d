"""Reflecting directions of fewer cells than ghost layers: a mirror image that
lies beyond the opposite side goes through that side's boundary, so no ghost
cell depends on the order in which a launch's threads write.  States and ghost
cells are the oracle's, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1711_06203_amd import workloads as W

pytestmark = pytest.mark.gpu

P, O, R, I = W.BC_PERIODIC, W.BC_OUTFLOW, W.BC_REFLECT, W.BC_INFLOW


@pytest.fixture(scope="module")
def ctx():
    from paper_1711_06203_amd import ctuppm
    c = ctuppm.Context()
    yield c
    c.set_fused(1)
    c.close()


@pytest.mark.parametrize("form", ["per_box", "batched", "graph", "waves"])
@pytest.mark.parametrize("n,box,bc_lo,bc_hi", [
    ((20, 1, 9), (20, 1, 9), (P, R, P), (P, R, P)),
    ((20, 1, 1), (7, 1, 1), (O, R, R), (O, R, R)),      # a tube of one cell across
    ((9, 8, 2), (9, 8, 2), (P, P, R), (P, P, O)),
    ((9, 8, 3), (5, 8, 2), (O, P, R), (R, P, R)),
    ((3, 9, 8), (2, 9, 4), (R, P, O), (I, P, R)),
    ((2, 3, 12), (1, 3, 5), (I, R, P), (R, R, P)),
    ((3, 3, 3), (3, 3, 3), (R, R, R), (R, R, R)),
])
def test_thin_reflecting_directions(ctx, form, n, box, bc_lo, bc_hi):
    from paper_1711_06203_amd import ctuppm
    scheme = (n[0] + n[2]) % 3
    prob = W.kelvin_helmholtz(n=n, box=box, seed=6, nspec=1)
    rng = np.random.default_rng(3)
    prob.U0 = prob.U0 * (1.0 + 0.05 * rng.random(prob.U0.shape))
    prob.scheme, prob.bc_lo, prob.bc_hi = scheme, bc_lo, bc_hi
    prob.inflow, prob.inflow_X = (1.25, 0.5, -0.25, 0.125, 2.0), (0.25,)
    ghosts = oracle.fill_domain(oracle.grow(prob.U0), oracle.params_of(prob))
    ref, dts, _ = oracle.run_problem(prob, 3)
    assert np.isfinite(ref).all()
    for fused in (1, 0):
        ctx.set_fused(fused)
        s = ctuppm.Solver(ctx, prob, form=form)
        s.step(1)
        U = s.UA.cpu().numpy()
        for (lo, hi), off, shape in zip(prob.boxes, s.lv[0]["offsets"], s.lv[0]["shapes"]):
            cells = (slice(None),) + tuple(slice(lo[d], hi[d] + 9) for d in (2, 1, 0))
            assert np.array_equal(U[off:off + int(np.prod(shape))].reshape(shape), ghosts[cells])
        s.step(2)
        assert np.array_equal(s.state(), ref) and s.dt() == dts[-1]
        s.close()
