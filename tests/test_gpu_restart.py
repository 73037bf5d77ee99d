"""A handle that is given a new initial field starts a new run: nothing of the
run before it (its ring of past levels, its history) may count. The first run
is filled with NaN, so that any value of it that is still multiplied, even by
a weight of zero, shows; the second must equal a fresh handle's run bit for
bit. PE edges down to twice the half-width (strips that overlap), a single PE,
the PE-major 3-D layout, the single-level schemes and Heun's second ring."""
import math

import numpy as np
import pytest
import torch

from tests._cases import initial_field, solver_for

pytestmark = pytest.mark.gpu

CASES = [
    # ndim, n, pe, order, integrator, scheme, L
    (1, (24,), (6,), 4, "ab2", "time", 4),
    (1, (13,), (1,), 6, "ab3", "time", 8),
    (1, (4096,), (64,), 4, "ab2", "time", 8),
    (2, (30, 18), (5, 3), 6, "rk2", "time", 8),
    (2, (42, 26), (3, 2), 2, "euler", "space222", 3),
    (2, (36, 40), (3, 4), 2, "euler", "nonuniform212", 4),
    (3, (20, 15, 12), (2, 1, 2), 4, "ab2", "time", 4),
    (3, (64, 32, 48), (2, 1, 2), 6, "rk2", "time", 8),
    (3, (32, 64, 8), (1, 2, 2), 4, "ab3", "time", 3),
    (3, (64, 32, 32), (2, 1, 1), 2, "euler", "space212", 3),
]


@pytest.mark.parametrize("ndim,n,pe,order,integrator,scheme,L", CASES)
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_new_state_leaves_nothing_of_the_run_before(ndim, n, pe, order, integrator, scheme, L, precision):
    dx = 2 * math.pi / max(n)
    r = {2: 0.05, 4: 0.005, 6: 0.002}[order]
    case = dict(ndim=ndim, n=n, pe=pe, order=order, integrator=integrator, equation="advdiff",
                c=(0.6, -0.3, 0.4)[:ndim], alpha=0.1, L=L, T=0, mode="rng", seed=7, scheme=scheme,
                dt=min(r * dx * dx / 0.1, 0.02 * dx), steps=L + 4, ic_seed=3)
    print(f"[restart] {case} {precision}", flush=True)
    u0 = torch.from_numpy(initial_field(case))
    fresh = solver_for(case, precision)
    fresh.set_state(u0)
    fresh.step(case["steps"])
    want = fresh.state()
    s = solver_for(case, precision)
    s.set_state(torch.full_like(u0, float("nan")))
    s.step(2 * L + 3)
    s.set_state(u0)
    s.step(case["steps"])
    got = s.state()
    assert bool(torch.isfinite(want).all())
    assert torch.equal(got, want)


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_new_ensemble_state_leaves_nothing_of_the_run_before(precision):
    from paper_1702_00496_amd import Ensemble
    members, fields = [], []
    for i, (n, pe, order, integ, L, mode) in enumerate([
            (64, 8, 2, "euler", 3, "rng"), (62, 2, 4, "ab2", 8, "rng"), (36, 6, 6, "ab2", 4, "rng"),
            (4096, 64, 4, "ab2", 8, "rng"), (1024, 16, 2, "euler", 4, "sync"), (20, 4, 2, "ab2", 1, "zero"),
            (15, 5, 2, "euler", 2, "rng"), (16384, 256, 4, "ab2", 8, "rng")]):
        dx = 2 * math.pi / n
        members.append(dict(n=n, pe=pe, order=order, integrator=integ, L=L, mode=mode, c=0.7, alpha=0.1,
                            dt=min({2: 0.05, 4: 0.005, 6: 0.002}[order] * dx * dx / 0.1, 0.02 * dx), seed=91 + i))
        x = np.arange(n) * dx
        fields.append(np.sin(x + 0.1 * i) + 0.5 * np.cos(2 * x))
    u0 = torch.from_numpy(np.concatenate(fields))
    fresh = Ensemble(members, precision=precision)
    fresh.set_state(u0)
    fresh.run(14)
    want = fresh.state()
    e = Ensemble(members, precision=precision)
    e.set_state(torch.full_like(u0, float("nan")))
    e.run(19)
    e.set_state(u0)
    e.run(14)
    assert bool(torch.isfinite(want).all())
    assert torch.equal(e.state(), want)
