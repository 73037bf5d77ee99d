"""The 1-D / 2-D stage kernel of the adjoint at the PE shapes and delay models
where its layout can go wrong, against the oracle's gradients at the bars of
test_gpu_adjoint.py: odd and even x edges, edges of twice the half-width, one
PE on an axis, more frame items than threads, more points than a thread loads
ahead, one to four levels, long delays, every delay mode, both equations, one or
two mu terms; and a plane too large for LDS (the strip and stage kernels).
dJ/dalpha is checked in FP64: on these inputs (white seeds, thousands of points
on an axis) it is the small remainder of mu times the Laplacian of the stored
levels, whose FP32 rounding grows as 1/dx^2 and has no bound relative to it."""
import math

import pytest
import torch

from tests._cases import field_errors, initial_field, oracle_for
from tests.test_gpu_adjoint import _gpu_grads, _oracle_grads, _say, _seed

pytestmark = pytest.mark.gpu

# n, pe, order, integrator, equation, L, T, mode, steps, every
CASES = [
    ((14, 12), (2, 2), 6, "rk2", "burgers", 8, 0, "rng", 14, 5),
    ((15, 8), (3, 2), 4, "ab2", "advdiff", 4, 0, "rng", 9, 4),
    ((4, 6), (2, 3), 2, "euler", "burgers", 3, 0, "rng", 8, 3),
    ((33, 24), (1, 2), 4, "rk2", "advdiff", 8, 0, "rng", 12, 20),
    ((128, 64), (2, 1), 6, "ab2", "burgers", 8, 0, "rng", 12, 5),        # 64 x 64
    ((65, 63), (1, 1), 4, "ab2", "advdiff", 3, 0, "rng", 5, 2),          # 65 x 63: a third pair per thread
    ((8, 1000), (1, 2), 4, "ab2", "burgers", 3, 0, "rng", 5, 2),         # 8 x 500
    ((4, 4096), (1, 4), 4, "rk2", "burgers", 2, 0, "rng", 3, 2),         # 4 x 1024 (FP64: too large for LDS)
    ((24, 18), (2, 3), 4, "ab2", "burgers", 4, 1, "rng", 9, 3),
    ((24, 18), (2, 2), 6, "rk2", "advdiff", 3, 2, "rng", 8, 4),
    ((24, 16), (2, 2), 4, "ab2", "burgers", 4, 0, "zero", 7, 3),
    ((22, 18), (2, 2), 6, "rk2", "burgers", 1, 0, "sync", 6, 2),
    ((4096,), (1,), 6, "ab2", "advdiff", 8, 0, "rng", 12, 5),
    ((35,), (5,), 6, "rk2", "burgers", 8, 0, "rng", 13, 4),
    ((27,), (3,), 4, "ab2", "advdiff", 4, 2, "rng", 9, 4),
    ((10,), (2,), 4, "rk2", "advdiff", 1, 0, "sync", 6, 4),
]


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "x".join(map(str, s[0])) + f"-{s[2]}-{s[3]}-{s[4]}-{s[7]}")
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_stage_kernel_matches_oracle_gradients(spec, precision):
    n, pe, order, integrator, equation, L, T, mode, steps, every = spec
    dx = 2 * math.pi / max(n)
    case = dict(ndim=len(n), n=n, pe=pe, order=order, integrator=integrator, equation=equation, c=(0.6, -0.4)[:len(n)],
                alpha=0.1, L=L, T=T, mode=mode, seed=13, steps=steps, every=every,
                dt=min({2: 0.05, 4: 0.01, 6: 0.002}[order] * dx * dx / 0.1, 0.02 * dx))
    _say(f"[adj2d] {spec} {precision}")
    u0, seed = initial_field(case), _seed(case)
    gu_o, ga_o = _oracle_grads(case, u0, seed)
    _, gu, ga = _gpu_grads(case, u0, seed, precision)
    tol = 1e-12 if precision == "f64" else 1e-5
    errs = field_errors(gu, gu_o, oracle_for(case, u0).prob)
    _say(f"[adj2d]   {errs} dalpha {ga:.9e} vs {ga_o:.9e}")
    assert all(v <= tol for v in errs.values()), errs
    if precision == "f64":
        assert ga == pytest.approx(ga_o, rel=tol)
