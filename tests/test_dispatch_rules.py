"""The rules that choose kernels, evaluated on the host."""
import pytest

from tests import _rules


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return _rules.build(str(tmp_path_factory.mktemp("rules")))


def test_3d_adjoint_kernel_follows_the_faster_one(rules):
    from tests.test_gpu_adjoint_choice3d import FEW, WIDE
    for want, cases in ((3, WIDE), (0, FEW)):
        for n, pe, order, integrator, equation, *_, precisions in cases:
            for precision in precisions.split():
                got = _rules.adjoint_kernel(rules, n, pe, order, integrator, equation, precision)
                assert got == want, (n, pe, order, equation, precision)
    # microseconds a stage (AB2) measured with the plane-walking kernel and with the strip and stage kernels
    for edges, pe, order, equation, precision, walk, spread in [
            ((24, 24, 96), (2, 2, 1), 4, "advdiff", "f64", 191, 31), ((24, 24, 96), (2, 2, 1), 6, "burgers", "f64", 685, 43),
            ((32, 32, 32), (2, 2, 2), 6, "burgers", "f32", 108, 41), ((32, 32, 32), (8, 8, 4), 6, "burgers", "f64", 363, 1010),
            ((32, 32, 32), (8, 8, 8), 6, "burgers", "f32", 217, 1743), ((64, 32, 32), (2, 2, 2), 4, "advdiff", "f32", 227, 43),
            ((64, 32, 32), (4, 8, 8), 4, "advdiff", "f64", 752, 1282), ((6, 6, 6), (16, 16, 16), 4, "advdiff", "f32", 166, 112),
            ((18, 18, 18), (8, 8, 8), 2, "advdiff", "f32", 40, 96), ((12, 12, 12), (8, 8, 8), 6, "burgers", "f64", 117, 156)]:
        n = [a * b for a, b in zip(edges, pe)]
        got = _rules.adjoint_kernel(rules, n, pe, order, "ab2", equation, precision)
        assert got == (3 if walk < spread else 0), (edges, pe, order, precision)
    # the cross-sections the plane-walking kernel cannot take, and the other dimensions
    assert _rules.adjoint_kernel(rules, (384, 384, 64), (8, 8, 16), 4, "ab2", "advdiff", "f32") == 0
    assert _rules.adjoint_kernel(rules, (1024, 1024), (16, 16), 4, "ab2", "advdiff", "f32") == 2
    assert _rules.adjoint_kernel(rules, (4096,), (1,), 6, "ab2", "burgers", "f64") == 2
