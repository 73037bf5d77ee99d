"""The 3-D stage kernel of the adjoint at the PE shapes and delay models where
its layout can go wrong, against the oracle's gradients at the bars of
test_gpu_adjoint.py (FP64 1e-12, FP32 1e-5 for dJ/du0 and 1e-4 for dJ/dalpha):
odd and even x edges, edges of twice the half-width, a single PE on an axis,
more frame items than points, the largest cross-section it takes and one it
does not, one to four levels, long delays (more entries of the g ring a value
than are read ahead), every delay mode, both equations, one or two mu terms,
segments longer than the run. And a run continued after the adjoint: the
context is at step N with its rings and its history."""
import math

import pytest
import torch

from tests._cases import field_errors, initial_field, oracle_for, solver_for
from tests.test_gpu_adjoint import _gpu_grads, _oracle_grads, _say, _seed

pytestmark = pytest.mark.gpu

# n, pe, order, integrator, equation, L, T, mode, steps, every
CASES = [
    ((14, 12, 12), (2, 2, 2), 6, "rk2", "burgers", 8, 0, "rng", 14, 5),
    ((10, 9, 8), (2, 1, 2), 4, "ab2", "advdiff", 4, 0, "rng", 9, 4),
    ((4, 4, 4), (2, 2, 2), 2, "euler", "burgers", 3, 0, "rng", 8, 3),
    ((33, 8, 12), (1, 2, 3), 4, "rk2", "advdiff", 8, 0, "rng", 12, 20),
    ((12, 66, 6), (2, 1, 1), 6, "ab2", "burgers", 4, 0, "rng", 6, 2),
    ((12, 12, 12), (2, 2, 2), 4, "ab2", "burgers", 4, 1, "rng", 9, 3),
    ((18, 12, 12), (3, 2, 1), 6, "rk2", "advdiff", 3, 2, "rng", 8, 4),
    ((24, 16, 8), (2, 2, 1), 4, "ab2", "burgers", 4, 0, "zero", 7, 3),
    ((22, 18, 14), (2, 2, 1), 6, "rk2", "burgers", 1, 0, "sync", 6, 2),
    ((30, 20, 12), (2, 2, 2), 4, "ab2", "advdiff", 1, 0, "sync", 6, 4),
    ((64, 64, 16), (2, 2, 2), 4, "euler", "burgers", 8, 0, "rng", 11, 4),
    ((64, 32, 8), (1, 1, 2), 2, "ab2", "advdiff", 3, 0, "rng", 6, 3),     # 64 x 32: 1024 threads
    ((48, 48, 8), (1, 1, 1), 4, "ab2", "burgers", 3, 0, "rng", 5, 2),     # 48 x 48: strip and stage kernels
]


def _case(n, pe, order, integrator, equation, L, T, mode, steps, every):
    dx = 2 * math.pi / max(n)
    r = {2: 0.05, 4: 0.01, 6: 0.002}[order]
    return dict(ndim=3, n=n, pe=pe, order=order, integrator=integrator, equation=equation, c=(0.6, -0.4, 0.3), alpha=0.1,
                L=L, T=T, mode=mode, seed=13, steps=steps, every=every, dt=min(r * dx * dx / 0.1, 0.02 * dx))


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "x".join(map(str, s[0])) + f"-{s[2]}-{s[3]}-{s[4]}-{s[7]}")
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_stage_kernel_matches_oracle_gradients(spec, precision):
    case = _case(*spec)
    _say(f"[adj3d] {spec} {precision}")
    u0, seed = initial_field(case), _seed(case)
    gu_o, ga_o = _oracle_grads(case, u0, seed)
    s, gu, ga = _gpu_grads(case, u0, seed, precision)
    tol = 1e-12 if precision == "f64" else 1e-5
    errs = field_errors(gu, gu_o, oracle_for(case, u0).prob)
    _say(f"[adj3d]   {errs} dalpha {ga:.9e} vs {ga_o:.9e}")
    assert all(v <= tol for v in errs.values()), errs
    assert ga == pytest.approx(ga_o, rel=tol if precision == "f64" else 1e-4)
    s.step(9)
    ref = solver_for(case, precision)
    ref.set_state(torch.from_numpy(u0))
    ref.step(case["steps"] + 9)
    assert s.n_step == ref.n_step
    assert torch.equal(s.state(), ref.state())


@pytest.mark.parametrize("n,pe,integrator", [((40, 36), (4, 3), "ab2"), ((40, 36), (2, 1), "rk2"), ((64,), (4,), "ab2"),
                                             ((36000,), (90,), "euler")])
def test_a_run_goes_on_after_the_adjoint(n, pe, integrator):
    dx = 2 * math.pi / max(n)
    case = dict(ndim=len(n), n=n, pe=pe, order=4, integrator=integrator, equation="advdiff", c=(0.6, -0.4)[:len(n)],
                alpha=0.1, L=4, T=0, mode="rng", seed=3, steps=11, every=4, dt=0.01 * dx * dx / 0.1)
    u0, seed = initial_field(case), _seed(case)
    s, _, _ = _gpu_grads(case, u0, seed, "f64")
    s.step(9)
    ref = solver_for(case, "f64")
    ref.set_state(torch.from_numpy(u0))
    ref.step(20)
    assert torch.equal(s.state(), ref.state())
