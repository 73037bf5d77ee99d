"""Long segments: the adjoint's scratch stays within 24 GiB of what the stored
levels and rings of L + T slots take. The reversal then puts the older levels back
into the segment's ring as it goes; gradients must equal those of short segments,
whose ring holds every level, bit for bit: through both 3-D kernel families and
field layouts, 2-D and 1-D, one and two rings, two level sets, several segments."""
import ctypes
import math

import pytest
import torch

from tests._cases import initial_field, solver_for
from tests.test_gpu_adjoint import _gpu_grads, _seed

pytestmark = pytest.mark.gpu

# n, pe, order, integrator, equation, precision, steps, long intervals, short interval
CASES = [
    ((1024, 1024), (128, 128), 6, "ab2", "advdiff", "f64", 6300, (2100,), 300),
    ((96, 96, 96), (16, 16, 16), 6, "rk2", "burgers", "f64", 1290, (640,), 100),
    ((128, 128, 128), (4, 4, 16), 6, "rk2", "burgers", "f32", 2840, (1420,), 200),
    ((1 << 20,), (1 << 18,), 4, "ab2", "burgers", "f64", 3150, (3140,), 400),
]


def _scratch(s, steps, every):
    v = ctypes.c_size_t(0)
    assert s._lib.at_adjoint_scratch_size(s._ctx, steps, every, ctypes.byref(v)) == 0
    return v.value


@pytest.mark.parametrize("n,pe,order,integrator,equation,precision,steps,intervals,short", CASES,
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_long_segments(n, pe, order, integrator, equation, precision, steps, intervals, short):
    dx, L, nd = 2 * math.pi / max(n), 8, len(n)
    case = dict(ndim=nd, n=n, pe=pe, order=order, integrator=integrator, equation=equation, c=(0.6, -0.4, 0.3)[:nd],
                alpha=0.1, L=L, T=0, mode="rng", seed=5, steps=steps,
                dt=min({4: 0.005, 6: 0.002}[order] * dx * dx / 0.1, 0.02 * dx))
    u0, seed = initial_field(case), _seed(case)
    s = solver_for(case, precision)
    field, w, rk2 = u0.size * (8 if precision == "f64" else 4), order // 2, integrator == "rk2"
    edges = [a // b for a, b in zip(n, pe)]
    slot = sum(2 * w * field // e for e in edges)
    rings = (2 if rk2 else 1) * (L + w + 1) * slot
    for every in intervals:
        levels = (every + 1) * field + (every * field if rk2 else 0)
        sets = 2 if levels + rings <= 4 << 30 else 1
        segments = -(-steps // every)
        # checkpoints, level sets, the last segment's start, adjoint fields and rings (in double where the strips are summed)
        need = (segments - 1) * (2 * field + rings) + sets * (levels + rings) + rings + 4 * field + 2 * rings + slot
        more = sets * (2 if rk2 else 1) * every * slot
        got = _scratch(s, steps, every)
        print(f"[scratch] {n} every {every}: {got / 2 ** 30:.2f} GiB, rings of every level {more / 2 ** 30:.2f}", flush=True)
        assert more > 24 << 30
        assert got <= need + (24 << 30)
    del s
    s, gu, ga = _gpu_grads(case, u0, seed, precision, every=short)
    del s
    torch.cuda.empty_cache()
    for every in intervals:
        print(f"[scratch] {n} every {every} {precision}", flush=True)
        s, gl, gal = _gpu_grads(case, u0, seed, precision, every=every)
        assert torch.equal(gl, gu) and gal == ga, every
        assert s.n_step == steps and bool(torch.isfinite(gl).all())
        del s
        torch.cuda.empty_cache()
