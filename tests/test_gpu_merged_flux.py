"""The flux stages that take the three directions in one launch, at the sizes
where their work lists can go wrong: boxes one cell thin along each axis,
ragged tails, planes just under and over a work unit, more problems than one
launch holds.  Every cell takes the same arithmetic as in the one-kernel-per-
direction stages, so states and counters are compared bit for bit (no
tolerance), and with the oracle."""
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


def _run(ctx, prob, steps, form, fused):
    from paper_1711_06203_amd import ctuppm
    ctx.set_fused(fused)
    s = ctuppm.Solver(ctx, prob, form=form)
    s.step(steps)
    out, cnt = s.state(), s.counters()
    s.close()
    return out, cnt


@pytest.mark.parametrize("form", ["per_box", "batched", "graph", "waves"])
@pytest.mark.parametrize("n,box", [
    ((12, 10, 8), (1, 10, 8)),      # one cell thin along x, y, z
    ((10, 12, 8), (10, 1, 8)),
    ((8, 10, 12), (8, 10, 1)),
    ((14, 15, 6), (14, 15, 6)),     # a halo-1 plane of 272 cells: just over one unit
    ((14, 14, 5), (14, 14, 5)),     # 256 cells: exactly one
    ((67, 9, 7), (64, 9, 7)),       # a three-cell tail beside a long box
    ((5, 70, 9), (5, 64, 4)),
])
def test_thin_and_ragged_boxes(ctx, form, n, box):
    prob = W.kelvin_helmholtz(n=n, box=box, seed=3, nspec=1)
    got, cnt = _run(ctx, prob, 2, form, 1)
    split, cnts = _run(ctx, prob, 2, form, 0)
    ref, _, _ = oracle.run_problem(prob, 2)
    assert np.array_equal(got, split) and np.array_equal(got, ref)
    assert np.array_equal(cnt, cnts)


@pytest.mark.parametrize("scheme,riemann", [(0, 0), (0, 1), (1, 0), (2, 1)])
def test_walls_and_solvers(ctx, scheme, riemann):
    prob = W.rayleigh_taylor(n=(24, 17, 20), seed=5, boxes=W.regular_boxes((24, 17, 20), (9, 8, 7)))
    prob.scheme, prob.riemann = scheme, riemann
    got, cnt = _run(ctx, prob, 2, "batched", 1)
    split, cnts = _run(ctx, prob, 2, "batched", 0)
    ref, _, _ = oracle.run_problem(prob, 2)
    assert np.array_equal(got, split) and np.array_equal(got, ref)
    assert np.array_equal(cnt, cnts)


def test_more_problems_than_one_launch_holds(ctx):
    from paper_1711_06203_amd import ctuppm
    ctx.set_fused(1)
    probs = [W.serving_request(seed=s, n=5 + s % 7) for s in range(19)]
    solvers = [ctuppm.Solver(ctx, p, form="batched") for p in probs]
    ctx.step(solvers, "batched", 2)
    for s, p in zip(solvers, probs):
        ref, _, _ = oracle.run_problem(p, 2)
        assert np.array_equal(s.state(), ref), p.n
        s.close()


@pytest.mark.parametrize("form,box", [("batched", 1), ("graph", 0), ("per_box", 2), ("waves", 2)])
def test_mol_dump_of_fluxes_kept_out_of_memory(ctx, form, box):
    """Without species the method of lines solves its normal fluxes inside the
    update; a stage dump still returns them, for the box that used the scratch last."""
    from paper_1711_06203_amd import ctuppm
    prob = W.rayleigh_taylor(n=(16, 12, 21), seed=5, boxes=W.regular_boxes((16, 12, 21), (16, 12, 7)))
    prob.scheme, prob.riemann = 1, 1
    ctx.set_wave_boxes(2)
    got = {}
    for fused in (1, 0):
        ctx.set_fused(fused)
        s = ctuppm.Solver(ctx, prob, form=form)
        s.step(2)
        before = s.counters()
        got[fused] = [s.stage_array(box, f"fn{d}", form=form) for d in range(3)]
        assert np.array_equal(before, s.counters())
        s.close()
    ctx.set_wave_boxes(64)
    for d in range(3):
        face = [slice(None)] * 4
        face[3 - d] = slice(1, None)  # faces 0..n; the slot below holds none
        assert np.array_equal(got[1][d][tuple(face)], got[0][d][tuple(face)])
