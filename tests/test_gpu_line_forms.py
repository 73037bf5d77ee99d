"""Ensemble members in every form a kept line has at 1024 threads (points per
thread, whole or short chunks, ring in LDS or in device memory, AB2 history in
registers or in device memory) and streamed: against the oracle element by
element (relative L2 and Linf <= 1e-12 FP64, <= 1e-5 FP32), and bit for bit across
runs cut so that some calls stream and some keep the members, and across
schedules. Which member takes which form is pinned on the host in
test_dispatch_rules.py."""
import math

import numpy as np
import pytest
import torch

from tests._cases import check_field

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}

# n, pe, order, integrator, L, mode, {precision: (points per thread, chunks a PE, short chunks, ring in memory, history too)}
MEMBERS = [
    (32768, 1024, 4, "ab2", 8, "rng", {"f32": (32, 1, 0, 1, 0), "f64": (32, 1, 0, 1, 1)}),
    (32768, 1024, 4, "euler", 4, "rng", {"f32": (32, 1, 0, 1, 0), "f64": (32, 1, 0, 1, 0)}),
    (32768, 512, 6, "ab2", 2, "rng", {"f32": (32, 2, 0, 0, 0), "f64": (32, 2, 0, 1, 1)}),
    (16384, 512, 4, "ab2", 8, "rng", {"f32": (32, 1, 0, 0, 0), "f64": (16, 2, 0, 1, 0)}),
    (16384, 1024, 6, "ab2", 8, "rng", {"f32": (16, 1, 0, 1, 0), "f64": (16, 1, 0, 1, 0)}),
    (15360, 1024, 4, "euler", 8, "rng", {"f32": (16, 1, 1, 1, 0), "f64": (16, 1, 1, 1, 0)}),
    (31744, 1024, 4, "euler", 8, "rng", {"f32": (32, 1, 1, 1, 0), "f64": (32, 1, 1, 1, 0)}),
    (65536, 512, 2, "ab2", 4, "rng", {"f32": (64, 2, 0, 0, 1), "f64": (0, 0, 0, 0, 0)}),
    (65536, 1024, 6, "euler", 2, "rng", {"f32": (64, 1, 0, 1, 0), "f64": (0, 0, 0, 0, 0)}),
    (8192, 128, 6, "euler", 3, "sync", {"f32": (32, 2, 0, 0, 0), "f64": (32, 2, 0, 0, 0)}),
    (100, 4, 4, "ab2", 8, "rng", {"f32": (4, 7, 3, 0, 0), "f64": (4, 7, 3, 0, 0)}),
]


def _members():
    members, fields = [], []
    for i, (n, pe, order, integ, L, mode, _) in enumerate(MEMBERS):
        dx = 2 * math.pi / n
        members.append(dict(n=n, pe=pe, order=order, integrator=integ, L=L, mode=mode, c=0.7, alpha=0.1, seed=41 + i,
                            dt=min({2: 0.05, 4: 0.005, 6: 0.002}[order] * dx * dx / 0.1, 0.02 * dx)))
        x = np.arange(n) * dx
        fields.append(np.sin(x + 0.1 * i) + 0.5 * np.cos(2 * x))
    return members, fields


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_every_form_of_a_member(precision):
    from oracle.solver import DelayModel, Oracle, Problem
    from paper_1702_00496_amd import Ensemble
    members, fields = _members()
    u0 = torch.from_numpy(np.concatenate(fields))
    steps = 23
    e = Ensemble(members, precision=precision)
    e.set_tuning(1, 1024)
    e.set_state(u0)
    e.run(steps)
    want = e.state()
    for groups, threads, cut in ((1, 1024, (1,) * 23), (1, 1024, (1, 20, 2)), (1, 512, (23,)), (4, 256, (2, 20, 1))):
        print(f"[forms] {groups} x {threads} {cut} {precision}", flush=True)
        e.set_tuning(groups, threads)
        e.set_state(u0)
        for k in cut:
            e.run(k)
        assert torch.equal(e.state(), want), (groups, threads, cut)
    for spec, m, field, got in zip(MEMBERS, members, fields, e.split(want.double().cpu())):
        print(f"[forms] {spec[:6]} {precision}", flush=True)
        o = Oracle(Problem(ndim=1, n=(m["n"],), pe=(m["pe"],), dt=m["dt"], order=m["order"], c=(0.7,), alpha=0.1,
                           integrator=m["integrator"]),
                   DelayModel(L=m["L"], mode=m["mode"], seed=m["seed"]), torch.from_numpy(field).reshape(1, 1, -1))
        o.run(steps)
        check_field(got.reshape(1, 1, -1), o, TOL[precision], label=(spec[:6], precision))
