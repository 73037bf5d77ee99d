"""dJ/dalpha of 1-D and 2-D problems in FP32, whose stage kernel takes the Laplacian
from sums of neighbours. On these inputs (white seeds) it is the small remainder of
dt sum mu (Laplacian of the stored levels): a level carries rounding of about
2^-24 max|u| times 1 + sqrt(steps), the Laplacian multiplies it by the sum of its
|taps|, and mu is a white field of unit variance or less, so that the error has a
standard deviation of at most dt steps sqrt(points) times that; six of them are
allowed."""
import math

import pytest

from tests._cases import initial_field
from tests.test_gpu_adjoint import _gpu_grads, _oracle_grads, _say, _seed
from tests.test_gpu_adjoint_stage2d import CASES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spec", CASES, ids=lambda s: "x".join(map(str, s[0])) + f"-{s[2]}-{s[3]}-{s[4]}-{s[7]}")
def test_alpha_gradient_in_fp32(spec):
    n, pe, order, integrator, equation, L, T, mode, steps, every = spec
    dx = 2 * math.pi / max(n)
    dt = min({2: 0.05, 4: 0.01, 6: 0.002}[order] * dx * dx / 0.1, 0.02 * dx)
    case = dict(ndim=len(n), n=n, pe=pe, order=order, integrator=integrator, equation=equation, c=(0.6, -0.4)[:len(n)],
                alpha=0.1, L=L, T=T, mode=mode, seed=13, steps=steps, every=every, dt=dt)
    u0, seed = initial_field(case), _seed(case)
    _, ga_o = _oracle_grads(case, u0, seed)
    _, _, ga = _gpu_grads(case, u0, seed, "f32")
    taps = {2: 4.0, 4: 16.0 / 3.0, 6: 6.0 + 2.0 / 45.0}[order]   # sum |c2| dx^2 of an axis
    lap = sum(taps * (v / (2 * math.pi)) ** 2 for v in n)
    sigma = dt * steps * math.sqrt(math.prod(n)) * 2.0 ** -24 * float(abs(u0).max()) * (1 + math.sqrt(steps)) * lap
    _say(f"[alpha2d] {spec} dalpha {ga:.9e} vs {ga_o:.9e}: {abs(ga - ga_o) / sigma:.2f} sigma, {sigma / abs(ga_o):.1e} of it")
    assert abs(ga - ga_o) <= 6 * sigma, (ga, ga_o, sigma)
