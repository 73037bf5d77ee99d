"""A 1-D context rounds alike whichever way it is stepped: as one launch that
keeps the line on its compute unit or as a sweep per step. Short calls of a large
state, and the levels an adjoint stores, come from the sweep; the run and the
gradient must not show it, bit for bit."""
import math

import pytest
import torch

from tests._cases import initial_field, solver_for
from tests.test_gpu_adjoint import _gpu_grads, _seed

pytestmark = pytest.mark.gpu


def _case(n, pe, order, integrator, equation, mode, L, steps):
    dx = 2 * math.pi / n
    return dict(ndim=1, n=(n,), pe=(pe,), order=order, integrator=integrator, equation=equation, c=(0.7,), alpha=0.1,
                L=L, T=0, mode=mode, seed=29, scheme="time", ic_seed=6, steps=steps,
                dt=min({2: 0.05, 4: 0.005, 6: 0.002}[order] * dx * dx / 0.1, 0.02 * dx))


# one and two steps of these are sweeps, the long call is one launch
CALLS = [
    (8192, 128, 2, "euler", "advdiff", "rng", 8),
    (8192, 128, 4, "ab2", "advdiff", "rng", 8),
    (8190, 182, 4, "ab2", "burgers", "rng", 4),        # PEs of 45: the scalar sweep
    (8192, 64, 4, "ab3", "burgers", "rng", 4),
    (7680, 80, 6, "ab3", "advdiff", "zero", 3),
    (8008, 91, 4, "ab3", "advdiff", "rng", 8),         # PEs of 88
    (7920, 99, 6, "rk2", "burgers", "rng", 3),
    (8184, 93, 2, "rk2", "advdiff", "rng", 8),
    (8192, 128, 4, "ab3", "burgers", "sync", 1),
    (8192, 128, 4, "ab2", "advdiff", "sync", 1),
]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("spec", CALLS, ids=lambda s: f"{s[0]}x{s[1]}-{s[2]}-{s[3]}-{s[4]}-{s[5]}")
def test_calls_of_any_length_give_the_same_run(spec, precision):
    case = _case(*spec, 17)
    print(f"[line calls] {spec} {precision}", flush=True)
    u0 = torch.from_numpy(initial_field(case))
    s = solver_for(case, precision)
    s.set_state(u0)
    s.step(17)
    want = s.state()
    assert bool(torch.isfinite(want).all())
    for cut in ((1,) * 17, (1, 9, 1, 2, 4), (10, 2, 1, 1, 3)):
        s.set_state(u0)
        for k in cut:
            s.step(k)
        assert torch.equal(s.state(), want), cut


GRADIENTS = [
    (252, 6, 4, "ab2", "burgers", "rng", 3),
    (96, 4, 6, "rk2", "burgers", "rng", 4),
    (27, 3, 6, "ab2", "advdiff", "rng", 8),            # 9 = 3 + 3 + 3
    (120, 8, 2, "euler", "burgers", "zero", 3),
    (1024, 16, 4, "rk2", "burgers", "sync", 1),
    (4096, 1024, 2, "ab2", "burgers", "rng", 4),
    (8192, 128, 4, "ab2", "burgers", "rng", 4),
]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("spec", GRADIENTS, ids=lambda s: f"{s[0]}x{s[1]}-{s[2]}-{s[3]}-{s[4]}-{s[5]}")
def test_gradient_of_a_line_is_that_of_the_run_it_returns(spec, precision):
    case = _case(*spec, 23)
    print(f"[line gradient] {spec} {precision}", flush=True)
    u0, seed = initial_field(case), _seed(case)
    ref = solver_for(case, precision)
    ref.set_state(torch.from_numpy(u0))
    ref.step(23)
    base = None
    for every in (1, 5, 23, 40):
        s, gu, ga = _gpu_grads(case, u0, seed, precision, every=every)
        assert torch.equal(s.state(), ref.state()), every
        base = base or (gu, ga)
        assert torch.equal(gu, base[0]) and ga == base[1], every


def test_a_long_call_is_several_launches():
    """40000 steps of a tiny line: three launches of at most 16384 steps (graph
    nodes of a captured call), the same bits as in short calls, and a replay goes
    on from the step the device holds."""
    import ctypes
    case = _case(16, 2, 2, "euler", "advdiff", "rng", 3, 40000)
    u0 = torch.from_numpy(initial_field(case))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ref = solver_for(case, "f64")
        ref.set_state(u0)
        for _ in range(80):
            ref.step(1000)
        s = solver_for(case, "f64")
        s.set_state(u0)
        s.step(0)
        side.synchronize()
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g, stream=side):
            s.step(40000)
        count = ctypes.c_size_t(0)
        hip = ctypes.CDLL("libamdhip64.so")
        assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(count)) == 0
        assert count.value == 3
        g.replay()
        s.step(40000)
        assert torch.equal(s.state(), ref.state())
