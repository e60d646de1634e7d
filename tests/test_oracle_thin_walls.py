"""Ghost cells of the oracle in directions of one to three cells with a
reflecting side: each is the image of a cell of the domain (or the inflow
state), found by following the boundaries from the ghost cell inwards."""
import itertools

import numpy as np
import pytest

import oracle
from paper_1711_06203_amd import workloads as W

O, R, I = W.BC_OUTFLOW, W.BC_REFLECT, W.BC_INFLOW


def source(c, n, lo, hi):
    """Cell (None: the inflow state) and sign of the normal momentum of ghost cell c."""
    sign = 1
    while not 0 <= c < n:
        bc = lo if c < 0 else hi
        if bc == I:
            return None, sign
        if bc == O:
            return (0 if c < 0 else n - 1), sign
        c, sign = (-1 - c if c < 0 else 2 * n - 1 - c), -sign
    return c, sign


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("d", [0, 1, 2])
@pytest.mark.parametrize("lo,hi", [p for p in itertools.product((O, R, I), repeat=2) if R in p])
def test_ghost_cells_of_a_thin_direction(n, d, lo, hi):
    e = [6, 5, 7]
    e[d] = n
    prob = W.kelvin_helmholtz(n=tuple(e), box=tuple(e), seed=4, nspec=1)
    prob.bc_lo = tuple(lo if x == d else W.BC_PERIODIC for x in range(3))
    prob.bc_hi = tuple(hi if x == d else W.BC_PERIODIC for x in range(3))
    prob.inflow, prob.inflow_X = (1.25, 0.5, -0.25, 0.125, 2.0), (0.25,)
    G = oracle.fill_domain(oracle.grow(prob.U0), oracle.params_of(prob))
    rho, u, v, w, p = prob.inflow
    inflow = np.array([rho, rho * u, rho * v, rho * w,
                       p * (1.0 / (prob.gamma - 1.0)) + 0.5 * rho * ((u * u + v * v) + w * w), rho * 0.25])
    valid = [slice(4, -4)] * 3
    for c in range(-4, n + 4):
        cells = list(valid)
        cells[2 - d] = c + 4
        got = G[(slice(None), *cells)]
        s, sign = source(c, n, lo, hi)
        if s is None:
            want = np.broadcast_to(inflow[:, None, None], got.shape).copy()
        else:
            cells[2 - d] = s + 4
            want = G[(slice(None), *cells)].copy()
        want[1 + d] *= sign
        assert np.array_equal(got, want), c
