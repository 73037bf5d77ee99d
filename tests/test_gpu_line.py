"""Ensemble members kept on one compute unit for all steps of a run, against the oracle element by element (relative L2 and
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

from tests._cases import check_field

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}

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
