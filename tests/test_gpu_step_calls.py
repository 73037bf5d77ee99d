"""The launches of one call carry their step number as an offset from the
device counter, which the last of them moves: however a run is cut into calls
and graph replays (one step, the chunk and a rest, two chunks, a call shorter
than the chunk, a reload in between), it must equal the run in one call bit for
bit, and the oracle. The PEs take the 1-D and 2-D sweeps over their tile edges
(fewer points than threads, more than two quads per thread, an x edge that is
not a multiple of 4), every integrator, the single-level and synchronous arms
and both 3-D paths."""
import math

import pytest
import torch

from tests._cases import check_field, initial_field, oracle_for, solver_for

pytestmark = pytest.mark.gpu

CASES = [
    # ndim, n, pe, order, integrator, scheme, L, mode
    (1, (9216,), (4,), 4, "ab2", "time", 4, "rng"),
    (1, (9000,), (4,), 2, "ab3", "time", 3, "rng"),
    (2, (8, 12), (2, 3), 4, "ab2", "time", 4, "rng"),
    (2, (128, 128), (2, 2), 4, "ab2", "time", 4, "rng"),
    (2, (60, 66), (1, 1), 6, "ab3", "time", 3, "rng"),
    (2, (88, 90), (2, 1), 4, "rk2", "time", 4, "rng"),
    (2, (84, 100), (2, 2), 4, "rk2", "time", 3, "rng"),
    (2, (66, 62), (1, 2), 2, "ab2", "time", 2, "rng"),
    (2, (150, 100), (2, 2), 6, "ab3", "time", 3, "rng"),
    (2, (42, 50), (2, 2), 4, "euler", "time", 3, "rng"),
    (2, (48, 40), (2, 2), 4, "ab2", "time", 1, "sync"),
    (2, (50, 42), (2, 2), 4, "ab3", "time", 1, "sync"),
    (2, (72, 80), (2, 2), 2, "euler", "space222", 3, "rng"),
    (2, (80, 72), (2, 2), 2, "ab2", "nonuniform212", 4, "rng"),
    (3, (24, 20, 12), (2, 2, 2), 4, "ab2", "time", 4, "rng"),
    (3, (64, 32, 8), (2, 1, 2), 4, "rk2", "time", 4, "rng"),
    (3, (32, 64, 8), (1, 2, 2), 4, "ab2", "time", 3, "rng"),
]


@pytest.mark.parametrize("ndim,n,pe,order,integrator,scheme,L,mode", CASES)
@pytest.mark.parametrize("precision,tol", [("f64", 1e-12), ("f32", 1e-5)])
def test_run_cut_into_calls_and_graphs(ndim, n, pe, order, integrator, scheme, L, mode, precision, tol):
    dx = 2 * math.pi / max(n)
    r = {2: 0.05, 4: 0.005, 6: 0.002}[order]
    case = dict(ndim=ndim, n=n, pe=pe, order=order, integrator=integrator, equation="advdiff",
                c=(0.6, -0.3, 0.4)[:ndim], alpha=0.1, L=L, T=0, mode=mode, seed=11, scheme=scheme,
                dt=min(r * dx * dx / 0.1, 0.02 * dx), steps=17, ic_seed=5)
    print(f"[calls] {case} {precision}", flush=True)
    u0 = torch.from_numpy(initial_field(case))
    whole = solver_for(case, precision)
    whole.set_state(u0)
    whole.step(17)
    s = solver_for(case, precision)
    s.set_state(u0)
    s.step(1)
    s.step(2)
    saved = s.save()
    s.set_graph(3)
    s.step(7)          # two replays and one launch
    s.load(saved)
    s.step(2)          # shorter than the graph
    s.step(6)          # two replays
    s.set_graph(0)
    s.step(6)
    assert torch.equal(s.state(), whole.state())
    o = oracle_for(case, u0.numpy())
    o.run(17)
    check_field(whole.state().double().cpu(), o, tol, label=(case, precision))
