"""1-D problems kept on one compute unit for all steps of a call: contexts
and ensemble members, against the oracle element by element (relative L2 and
Linf <= 1e-12 FP64, <= 1e-5 FP32) where the layout can go wrong: PE edges of one
chunk, of short chunks (one point less than the others) and of many, lines that
just fill a workgroup's threads, more faces than one batch of drawn delays
covers per step, every integrator, both equations, every delay mode and runs
across several batches of delays. Schedules and splits of a run must agree bit
for bit, also where one of them streams a member through the caches."""
import math

import numpy as np
import pytest
import torch

from tests._cases import check_field, initial_field, oracle_for, solver_for

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}

# n, pe, order, integrator, equation, mode, L, steps
CONTEXTS = [
    (4, 1, 4, "ab2", "advdiff", "rng", 4, 150),         # one chunk, its own neighbour
    (3, 1, 2, "euler", "advdiff", "rng", 2, 70),        # one short chunk
    (14, 2, 6, "rk2", "advdiff", "rng", 8, 20),         # 7 = 4 + 3
    (27, 3, 6, "ab3", "burgers", "rng", 3, 70),         # 9 = 3 + 3 + 3
    (62, 2, 4, "ab3", "advdiff", "rng", 8, 140),
    (252, 6, 4, "ab2", "burgers", "rng", 3, 130),
    (315, 5, 2, "rk2", "burgers", "zero", 3, 40),
    (200, 8, 4, "rk2", "advdiff", "sync", 1, 30),
    (96, 4, 4, "ab3", "advdiff", "host", 5, 60),
    (4096, 64, 2, "euler", "advdiff", "rng", 8, 12),    # 1024 chunks of four
    (8192, 128, 4, "ab2", "burgers", "rng", 4, 8),      # 1024 chunks of eight
    (4096, 1024, 2, "euler", "advdiff", "rng", 4, 9),   # 2048 faces: batches of two steps
    (8192, 2048, 2, "ab2", "advdiff", "rng", 3, 9),     # 4096 faces: batches of one step
    (1100, 220, 2, "ab2", "advdiff", "rng", 4, 9),      # PEs of 5: stepped launch by launch
    (10240, 160, 4, "ab2", "advdiff", "rng", 4, 6),     # too many points: launch by launch
]


def _case(n, pe, order, integrator, equation, mode, L, steps):
    dx = 2 * math.pi / n
    case = dict(ndim=1, n=(n,), pe=(pe,), order=order, integrator=integrator, equation=equation, c=(0.7,), alpha=0.1,
                L=L, T=0, mode=mode, seed=29, scheme="time", ic_seed=6, steps=steps,
                dt=min({2: 0.05, 4: 0.005, 6: 0.002}[order] * dx * dx / 0.1, 0.02 * dx))
    if mode == "host":
        case["host"] = np.random.Generator(np.random.PCG64(2)).integers(0, L, size=(steps, pe, 1, 2)).astype(np.int8)
    return case


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("spec", CONTEXTS, ids=lambda s: f"{s[0]}x{s[1]}-{s[2]}-{s[3]}-{s[4]}-{s[5]}")
def test_context_on_one_compute_unit_matches_the_oracle(spec, precision):
    case = _case(*spec)
    print(f"[line] {spec} {precision}", flush=True)
    u0 = initial_field(case)
    s = solver_for(case, precision)
    s.set_state(torch.from_numpy(u0))
    s.step(case["steps"])
    got = s.state()
    assert s.n_step == case["steps"]
    o = oracle_for(case, u0)
    o.run(case["steps"])
    check_field(got.double().cpu(), o, TOL[precision], label=(spec, precision))
    # the same run in pieces, through a checkpoint and as a graph
    s.set_state(torch.from_numpy(u0))
    s.set_graph(2)
    s.step(1)
    s.step(2)
    ck = s.save()
    s.step(case["steps"] - 3)
    assert torch.equal(s.state(), got)
    s.load(ck)
    for _ in range(3):
        s.step(1)
    s.step(case["steps"] - 6)
    assert torch.equal(s.state(), got)


# n, pe, order, integrator, L, mode
MEMBERS = [
    (65536, 1024, 4, "ab2", 8, "rng"),     # history and ring in device memory
    (65536, 1024, 4, "ab2", 2, "rng"),     # history in device memory
    (65536, 1024, 2, "euler", 8, "rng"),
    (32256, 512, 4, "ab2", 8, "rng"),      # 63 = 32 + 31
    (31744, 1024, 6, "ab2", 4, "rng"),     # PEs of 31
    (20480, 40, 4, "ab2", 4, "rng"),       # PEs of 512
    (16384, 128, 6, "euler", 3, "sync"),
    (3000, 60, 2, "ab2", 3, "rng"),        # 50 = 7 of 7 and 1
    (1024, 16, 2, "euler", 6, "rng"),
    (40, 4, 4, "ab2", 5, "zero"),
    (25, 5, 2, "euler", 2, "rng"),         # PEs of 5: streamed
]


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_long_and_short_members_agree_across_schedules_and_with_the_oracle(precision):
    from oracle.solver import DelayModel, Oracle, Problem
    from paper_1702_00496_amd import Ensemble
    members, fields = [], []
    for i, (n, pe, order, integ, L, mode) in enumerate(MEMBERS):
        dx = 2 * math.pi / n
        members.append(dict(n=n, pe=pe, order=order, integrator=integ, L=L, mode=mode, c=0.7, alpha=0.1, seed=17 + i,
                            dt=min({2: 0.05, 4: 0.005, 6: 0.002}[order] * dx * dx / 0.1, 0.02 * dx)))
        x = np.arange(n) * dx
        fields.append(np.sin(x + 0.1 * i) + 0.5 * np.cos(2 * x))
    u0 = torch.from_numpy(np.concatenate(fields))
    steps = 11
    e = Ensemble(members, precision=precision)
    e.set_state(u0)
    e.run(steps)
    want = e.state()
    for groups, threads in ((1, 1024), (1, 256), (2, 512), (4, 1024)):
        e.set_tuning(groups, threads)
        e.set_state(u0)
        e.run(4)
        e.run(1)
        e.run(steps - 5)
        assert torch.equal(e.state(), want), (groups, threads)
    for i, got in enumerate(e.split(want.double().cpu())):
        m = members[i]
        print(f"[line] member {MEMBERS[i]} {precision}", flush=True)
        o = Oracle(Problem(ndim=1, n=(m["n"],), pe=(m["pe"],), dt=m["dt"], order=m["order"], c=(0.7,), alpha=0.1,
                           integrator=m["integrator"]),
                   DelayModel(L=m["L"], mode=m["mode"], seed=m["seed"]), torch.from_numpy(fields[i]).reshape(1, 1, -1))
        o.run(steps)
        check_field(got.reshape(1, 1, -1), o, TOL[precision], label=(MEMBERS[i], precision))
