"""Stage dumps of the normal fluxes of a method-of-lines step without species,
which the update solves itself: a dump recomputes them from the face states,
where the step left these, whatever was set or bound again since.  The split
stages keep the fluxes in memory, so their dumps after the same calls are the
reference, bit for bit; nothing beyond the bound workspace is written."""
import ctypes

import numpy as np
import pytest

from paper_1711_06203_amd import workloads as W

pytestmark = pytest.mark.gpu
TAIL = 16 << 20  # allocated past the bound workspace, and watched


@pytest.fixture(scope="module")
def ctx():
    from paper_1711_06203_amd import ctuppm
    c = ctuppm.Context()
    yield c
    c.set_fused(1)
    c.set_wave_boxes(64)
    c.close()


def _bind(s, buf):
    s.ctx.call("ctuppm_bind_workspace", s.pid, ctypes.c_void_p(buf.data_ptr()), buf.numel() - TAIL)


def _after(ctx, prob, fused, form, wave, between, waves_then, boxes, room=None):
    """Two steps, then `between` under each wave size of waves_then, then the
    flux dumps of `boxes` (None where refused)."""
    from paper_1711_06203_amd import ctuppm
    ctx.set_fused(fused)
    ctx.set_wave_boxes(wave)
    s = ctuppm.Solver(ctx, prob, form=form)
    size = ctypes.c_size_t(s.ws.numel())
    if room:
        ctx.call("ctuppm_workspace_bytes", s.pid, ctuppm.FORMS[room], ctypes.byref(size))
    buf = ctx.torch.zeros((size.value + TAIL,), dtype=ctx.torch.uint8, device=s.dev)
    buf[-TAIL:] = 0x5A
    _bind(s, buf)
    s.step(2)
    for w in waves_then:
        ctx.set_wave_boxes(w)
        if between == "state":
            s._bind(0)
        elif between == "workspace":
            _bind(s, buf)
        elif between == "planes":
            ctx.set_stage_planes("riemann_xyz", 1)
    out = []
    for b in boxes:
        for d in range(3):
            try:
                out.append(s.stage_array(b, f"fn{d}", form=form))
            except ctuppm.CtuError as e:
                assert e.code == ctuppm.ENOMEM
                out.append(None)
    ctx.torch.cuda.synchronize()
    tail_kept = bool((buf[-TAIL:] == 0x5A).all())
    s.close()
    return out, tail_kept


@pytest.mark.parametrize("form", ["waves", "per_box", "batched"])
@pytest.mark.parametrize("between", ["nothing", "state", "workspace", "planes"])
@pytest.mark.parametrize("waves_then", [(3,), (2,), (5,), (64,), (2, 5), (5, 3)])
def test_flux_dumps_after_the_wave_size_changed(ctx, form, between, waves_then):
    prob = W.rayleigh_taylor(n=(16, 12, 21), seed=5, boxes=W.regular_boxes((16, 12, 21), (16, 12, 3)))
    prob.scheme = 1
    got, kept = _after(ctx, prob, 1, form, 3, between, waves_then, range(7))
    ref, _ = _after(ctx, prob, 0, form, 3, between, waves_then, range(7))
    assert kept
    assert any(r is not None and np.abs(r).max() > 0.0 for r in ref)
    for a, b in zip(got, ref):
        assert (a is None) == (b is None)
        if a is not None:
            assert np.array_equal(a, b)


@pytest.mark.parametrize("between", ["nothing", "state"])
def test_dump_of_a_small_box_beside_large_ones(ctx, between):
    """Waves of 4 boxes in a workspace that would hold them all, then waves of 5:
    box 4 (4^3) and box 9 (8 x 8 x 32) share a slot, where the fluxes of box 9
    would end past the workspace."""
    def slab(z, edges):  # boxes that tile the plane, from z on
        return [((x, y, z), (x + e[0] - 1, y + e[1] - 1, z + e[2] - 1)) for x, y, e in edges]
    large = [(0, 0, (8, 8, 32))]
    boxes = slab(0, large) + slab(32, large) + slab(64, large)
    boxes += slab(96, [(x, y, (4, 4, 4)) for y in (0, 4) for x in (0, 4)])
    boxes += slab(100, [(0, y, (8, 4, 1)) for y in (0, 4)]) + slab(101, large)
    prob = W.rayleigh_taylor(n=(8, 8, 133), seed=5, boxes=boxes)
    prob.scheme = 1
    got, kept = _after(ctx, prob, 1, "waves", 4, between, (5,), range(10), room="batched")
    ref, _ = _after(ctx, prob, 0, "waves", 4, between, (5,), range(10), room="batched")
    assert kept and all(g is not None for g in got[12:15]) and got[29] is None
    for a, b in zip(got[12:15] + got[27:], ref[12:15] + ref[27:]):  # slot 4: no box has used it
        assert (a is None) == (b is None) and (a is None or np.array_equal(a, b))
