"""The two-shock solver stops its Newton steps once they repeat.  Faces where
they settle at once (uniform states), where the last bits alternate (states a
few ulps apart), where all steps are needed (jumps of four decades) and waves
that hold all three are compared with the oracle, which takes every step: the
same bits."""
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
    c.close()


def _states(kind, n, seed):
    rng = np.random.default_rng(seed)
    shape = (n[2], n[1], n[0])
    base = rng.uniform(0.3, 3.0, 2)
    rho, p = np.full(shape, base[0]), np.full(shape, base[1])
    vel = [np.full(shape, v) for v in rng.uniform(-1.0, 1.0, 3)]
    where = {"uniform": 0.0, "ulps": 0.0, "jumps": 1.0, "mixed": 0.3}[kind]
    if kind in ("ulps", "mixed"):
        for a in (rho, p, *vel):
            a *= 1.0 + rng.integers(-3, 4, shape) * 2.0 ** -52
    jump = rng.random(shape) < where
    rho[jump] *= 10.0 ** rng.uniform(-2, 2, jump.sum())
    p[jump] *= 10.0 ** rng.uniform(-2, 2, jump.sum())
    for v in vel:
        v[jump] += rng.normal(0.0, 1.0, jump.sum())
    E = p / (1.4 - 1.0) + 0.5 * rho * (vel[0] ** 2 + vel[1] ** 2 + vel[2] ** 2)
    return np.stack([rho, rho * vel[0], rho * vel[1], rho * vel[2], E])


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("kind", ["uniform", "ulps", "jumps", "mixed"])
@pytest.mark.parametrize("n", [(17, 9, 8), (40, 12, 10)])
def test_bits_of_every_step(ctx, kind, n, scheme):
    from paper_1711_06203_amd import ctuppm
    for seed in range(4):
        prob = W.Problem("states", n, 1.4, _states(kind, n, 10 * seed + n[0]), W.regular_boxes(n, (n[0], n[1], 5)),
                         cfl=0.2, scheme=scheme, riemann=1, limiter=seed % 2)
        s = ctuppm.Solver(ctx, prob, form="batched")
        s.step(2)
        ref, dts, _ = oracle.run_problem(prob, 2)
        assert np.array_equal(s.state(), ref, equal_nan=True), seed
        assert np.array_equal(np.array([s.dt()]), np.array([dts[-1]]), equal_nan=True)
        s.close()
