"""dt and the commit taken by the last blocks of the conversion and of the update
against the launches of their own that the waves form keeps (same bits), up to
the largest sets that take them, where a problem's counters each count many
blocks; and a rejected step at those sizes, whose counters have to be ready for
the next one."""
import numpy as np
import pytest

from paper_1711_06203_amd import workloads as W

pytestmark = pytest.mark.gpu

P, O, R = W.BC_PERIODIC, W.BC_OUTFLOW, W.BC_REFLECT


@pytest.fixture(scope="module")
def ctx():
    from paper_1711_06203_amd import ctuppm
    c = ctuppm.Context()
    yield c
    c.close()


def _prob(n, box, scheme, bare, seed=5):
    prob = W.kelvin_helmholtz(n=n, box=box, seed=seed)
    prob.scheme = scheme
    if bare:  # a level whose ghosts are not all mapped: conversion in a launch of its own
        prob.boxes = prob.boxes[:-1]
        prob.bc_lo, prob.bc_hi = (O, P, P), (O, P, P)
    else:
        prob.bc_lo, prob.bc_hi = (O, P, R), (R, P, O)
    return prob


def _run(ctx, prob, form, steps):
    from paper_1711_06203_amd import ctuppm
    s = ctuppm.Solver(ctx, prob, form=form)
    s.UA[ctx.torch.isnan(s.UA) | (s.UA == 0.0)] = 0.125  # what bare parts hold
    out = []
    for _ in range(steps):
        s.step(1)
        out += [s.dt(), s.counters()]
    out += [s.UA.cpu().numpy(), s.UB.cpu().numpy(), s.current()]
    s.close()
    return out


SIZES = [
    ((62, 62, 50), (62, 62, 50), False),   # 800 update units
    ((90, 90, 63), (90, 90, 63), False),   # 2016
    ((90, 90, 63), (90, 90, 21), True),    # 1344 in boxes with bare ghost cells
    ((101, 101, 93), (101, 101, 93), False),  # 3720, 1.2 M cells with ghosts
    ((84, 72, 64), (16, 16, 16), False),   # 1536 in boxes of 16^3 and less
]


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("n,box,bare", SIZES)
def test_equal_to_launches_of_their_own(ctx, n, box, bare, scheme):
    prob = _prob(n, box, scheme, bare)
    ref = _run(ctx, prob, "waves", 3)
    for form in ("batched", "graph"):
        for a, b in zip(_run(ctx, prob, form, 3), ref):
            assert np.array_equal(a, b, equal_nan=True), form


@pytest.mark.parametrize("form", ["batched", "graph"])
@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("n,box", [((90, 90, 63), (90, 90, 63)), ((101, 101, 93), (101, 101, 93))])
def test_rejected_step(ctx, n, box, scheme, form):
    from paper_1711_06203_amd import ctuppm
    prob = _prob(n, box, scheme, False)
    s = ctuppm.Solver(ctx, prob, form="waves")
    s.step(3)
    ref = (s.state(), s.dt())
    s.close()
    s = ctuppm.Solver(ctx, prob, form=form)
    s.set_fail_hook(1)
    for _ in range(2):
        s.step_guarded(1)
        ctx.torch.cuda.synchronize()
    with pytest.raises(ctuppm.Rejected):
        s.step_guarded(1)
    assert s.rejections() == 1
    s.step_guarded(1)  # the hook fired once: the step is redone
    s.step_guarded(1)
    assert s.counters()[5] == 3 and s.dt() == ref[1]
    assert np.array_equal(s.state(), ref[0])
    s.close()
