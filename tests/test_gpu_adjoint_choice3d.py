"""3-D gradients on both sides of the rule that chooses the stage kernel
(adj3d_pays), against the oracle's: shapes with PEs enough for the plane-walking
kernel (its PE edges and threads where the layout can go wrong), and few or deep
PEs, which the strip and stage kernels take in both field layouts (32 x 32
cross-sections are kept PE after PE).

FP64 1e-12, FP32 1e-5 for dJ/du0 (the bars of test_gpu_adjoint.py). dJ/dalpha is
dt sum mu (Laplacian of the stored levels): a level carries rounding of about
2^-24 (FP64 2^-53) max|u| times 1 + sqrt(steps), the Laplacian multiplies it by
the sum of its |taps|, and mu is a white field of unit variance or less, so that
the error has a standard deviation of at most dt steps sqrt(points) times that;
six of them are allowed (FP64: twelve, the oracle rounds as well)."""
import math

import pytest
import torch

from tests._cases import field_errors, initial_field, oracle_for, solver_for
from tests.test_gpu_adjoint import _gpu_grads, _oracle_grads, _say, _seed

pytestmark = pytest.mark.gpu

# n, pe, order, integrator, equation, L, T, mode, steps, every, precisions
WIDE = [
    ((10, 9, 8), (2, 1, 2), 4, "ab2", "advdiff", 4, 0, "rng", 9, 4, "f32 f64"),
    ((33, 8, 8), (1, 2, 2), 4, "rk2", "advdiff", 8, 0, "rng", 12, 20, "f32 f64"),
    ((12, 66, 54), (2, 11, 9), 4, "ab2", "burgers", 4, 1, "rng", 9, 3, "f32 f64"),
    ((96, 112, 8), (8, 14, 1), 4, "ab2", "burgers", 4, 0, "zero", 7, 3, "f32 f64"),
    ((30, 40, 48), (2, 4, 8), 4, "ab2", "advdiff", 1, 0, "sync", 6, 4, "f32 f64"),
    ((64, 64, 24), (2, 2, 3), 4, "euler", "burgers", 8, 0, "rng", 11, 4, "f32 f64"),     # PE after PE
    ((14, 66, 66), (2, 11, 11), 6, "rk2", "burgers", 8, 0, "rng", 14, 5, "f32"),
    ((6, 132, 72), (1, 2, 12), 6, "ab2", "burgers", 4, 0, "rng", 6, 2, "f32"),            # more frame items than points
    ((48, 48, 96), (8, 8, 8), 6, "rk2", "advdiff", 3, 2, "rng", 4, 4, "f32"),
    ((44, 63, 98), (4, 7, 7), 6, "rk2", "burgers", 1, 0, "sync", 4, 2, "f32"),
    ((35, 42, 84), (5, 7, 14), 6, "rk2", "advdiff", 8, 0, "rng", 12, 5, "f64"),
    ((6, 396, 96), (1, 6, 16), 6, "ab2", "burgers", 4, 0, "rng", 5, 2, "f64"),
    ((26, 132, 130), (2, 11, 13), 6, "rk2", "burgers", 4, 0, "rng", 4, 4, "f64"),
    ((64, 32, 52), (1, 1, 13), 2, "ab2", "advdiff", 3, 0, "rng", 6, 3, "f32"),           # 64 x 32: 1024 threads
    ((64, 160, 40), (1, 5, 10), 2, "ab2", "advdiff", 3, 0, "rng", 6, 3, "f64"),
    ((64, 64, 60), (1, 2, 15), 4, "ab2", "burgers", 3, 0, "rng", 5, 2, "f32"),
]
FEW = [
    ((64, 32, 48), (2, 1, 3), 2, "ab2", "advdiff", 8, 0, "rng", 12, 5, "f32 f64"),       # PE after PE
    ((32, 64, 32), (1, 2, 1), 4, "rk2", "burgers", 4, 0, "rng", 8, 3, "f32 f64"),
    ((64, 64, 24), (2, 2, 1), 6, "ab2", "burgers", 3, 0, "rng", 6, 2, "f32 f64"),
    ((32, 32, 32), (1, 1, 2), 4, "ab2", "advdiff", 3, 2, "rng", 7, 3, "f32 f64"),
    ((32, 32, 24), (1, 1, 1), 6, "rk2", "advdiff", 4, 0, "zero", 5, 2, "f32 f64"),
    ((64, 32, 32), (2, 1, 1), 4, "euler", "burgers", 1, 0, "sync", 5, 2, "f32 f64"),
    ((48, 48, 96), (2, 2, 1), 4, "ab2", "advdiff", 4, 0, "rng", 5, 2, "f32 f64"),        # 24 x 24 x 96
    ((64, 64, 16), (1, 2, 2), 4, "rk2", "burgers", 3, 0, "rng", 4, 3, "f32 f64"),        # 64 x 32
]
CASES = [(c[:-1], p) for c in WIDE + FEW for p in c[-1].split()]


@pytest.mark.parametrize("spec,precision", CASES, ids=lambda v: v if isinstance(v, str) else
                         "x".join(map(str, v[0])) + f"-{v[2]}-{v[3]}-{v[4]}-{v[7]}")
def test_gradients_on_both_sides_of_the_choice(spec, precision):
    n, pe, order, integrator, equation, L, T, mode, steps, every = spec
    dx = 2 * math.pi / max(n)
    dt = min({2: 0.05, 4: 0.01, 6: 0.002}[order] * dx * dx / 0.1, 0.02 * dx)
    case = dict(ndim=3, n=n, pe=pe, order=order, integrator=integrator, equation=equation, c=(0.6, -0.4, 0.3), alpha=0.1,
                L=L, T=T, mode=mode, seed=13, steps=steps, every=every, dt=dt)
    _say(f"[choice3d] {spec} {precision}")
    u0, seed = initial_field(case), _seed(case)
    gu_o, ga_o = _oracle_grads(case, u0, seed)
    s, gu, ga = _gpu_grads(case, u0, seed, precision)
    tol = 1e-12 if precision == "f64" else 1e-5
    errs = field_errors(gu, gu_o, oracle_for(case, u0).prob)
    _say(f"[choice3d]   {errs} dalpha {ga:.9e} vs {ga_o:.9e}")
    assert all(v <= tol for v in errs.values()), errs
    taps = {2: 4.0, 4: 16.0 / 3.0, 6: 6.0 + 2.0 / 45.0}[order]   # sum |c2| dx^2 of an axis
    lap = sum(taps * (v / (2 * math.pi)) ** 2 for v in n)
    eps = 2.0 ** -24 if precision == "f32" else 2.0 ** -53
    sigma = dt * steps * math.sqrt(math.prod(n)) * eps * float(abs(u0).max()) * (1 + math.sqrt(steps)) * lap
    assert abs(ga - ga_o) <= (6 if precision == "f32" else 12) * sigma, (ga, ga_o, sigma)
    s.step(5)
    ref = solver_for(case, precision)
    ref.set_state(torch.from_numpy(u0))
    ref.step(steps + 5)
    assert torch.equal(s.state(), ref.state())
