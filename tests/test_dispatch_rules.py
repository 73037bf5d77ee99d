"""The rules that choose kernels, evaluated on the host."""
import ctypes

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


def test_short_calls_of_large_lines_take_the_sweep(rules):
    """Microseconds a call measured as one launch and as sweeps."""
    for n, pe, order, integrator, precision, steps, launch, sweeps in [
            (256, 8, 2, "euler", "f64", 1, 4.8, 6.1), (1024, 16, 4, "ab2", "f64", 1, 5.5, 6.2),
            (2048, 32, 4, "ab3", "f64", 1, 7.1, 5.8), (4096, 64, 4, "ab2", "f64", 1, 8.4, 6.3),
            (4096, 64, 4, "ab2", "f64", 2, 9.4, 11.5), (8192, 128, 4, "ab2", "f64", 1, 13.1, 6.3),
            (8192, 128, 4, "ab2", "f64", 2, 15.1, 11.6), (8192, 128, 4, "ab3", "f64", 3, 20.6, 17.3),
            (8192, 128, 2, "euler", "f32", 2, 7.2, 11.1), (8192, 128, 4, "rk2", "f32", 1, 9.8, 11.2),
            (4096, 8, 6, "rk2", "f64", 1, 16.0, 12.2), (1024, 16, 6, "rk2", "f64", 1, 8.6, 11.6),
            (8192, 8, 6, "rk2", "f32", 2, 14.9, 20.9)]:
        v = _rules.line(n, pe, order, integrator, 8, "rng")
        assert rules.context_pt(v, _rules.width(precision)) > 0
        assert rules.pays(v, _rules.width(precision), ctypes.c_longlong(steps)) == (launch < sweeps), (n, order, integrator, steps)
        assert rules.pays(v, _rules.width(precision), ctypes.c_longlong(50)) == 1


def test_short_ensemble_runs_are_streamed(rules):
    """Microseconds a run measured with every member kept and streamed."""
    for per_cu, n, pe, order, precision, steps, kept, streamed in [
            (1, 1024, 16, 2, "f64", 1, 17.0, 12.0), (1, 1024, 16, 4, "f32", 6, 18.7, 26.0),
            (1, 4096, 64, 4, "f64", 1, 23.0, 15.0), (1, 4096, 64, 4, "f64", 6, 29.0, 40.0),
            (1, 16384, 256, 4, "f64", 1, 62.0, 33.0), (1, 16384, 256, 4, "f64", 6, 75.0, 144.0),
            (2, 8192, 128, 4, "f64", 1, 81.0, 33.0), (2, 8192, 128, 4, "f64", 6, 97.0, 144.0),
            (2, 65536, 1024, 4, "f32", 1, 273.0, 109.0), (2, 65536, 1024, 4, "f32", 6, 418.0, 567.0),
            (1, 32768, 512, 4, "f64", 3, 209.0, 145.0), (1, 32768, 512, 4, "f64", 16, 529.0, 725.0)]:
        v = _rules.line(n, pe, order, "euler" if order == 2 else "ab2", 8, "rng")
        t = (ctypes.c_double * 2)()
        rules.ens(v, _rules.width(precision), per_cu, ctypes.c_longlong(steps), t)
        assert (t[1] < t[0]) == (streamed < kept), (n, order, precision, steps, list(t))


def test_plans_of_members_and_contexts(rules):
    from tests import test_gpu_line as G
    from tests.test_gpu_line_forms import MEMBERS
    out = (ctypes.c_int * 5)()
    for n, pe, order, integrator, L, mode, want in MEMBERS:
        for precision, form in want.items():
            rules.member_plan(_rules.line(n, pe, order, integrator, L, mode), _rules.width(precision), 1024, out)
            assert tuple(out) == form, (n, pe, order, integrator, precision, tuple(out))
    # points per thread of the contexts whose runs are compared with the oracle (0: a sweep per step)
    points = {(8192, 2048): 0, (1100, 220): 0, (10240, 160): 0, (4096, 64): 8, (8192, 128): 8}
    for n, pe, order, integrator, _, mode, L, _ in G.CONTEXTS:
        for precision in ("f64", "f32"):
            v = _rules.line(n, pe, order, integrator, L, mode)
            assert rules.context_pt(v, _rules.width(precision)) == points.get((n, pe), 4), (n, pe, precision)
    # overridden level counts, PEs of more threads than a workgroup, chunks shorter than the half-width
    assert rules.context_pt(_rules.line(64, 4, 4, "ab2", 4, "rng", T=2), 8) == 0
    assert rules.context_pt(_rules.line(4096, 1024, 2, "euler", 4, "rng"), 8) == 4
    assert rules.context_pt(_rules.line(4100, 1025, 2, "euler", 4, "rng"), 8) == 0
    assert rules.context_pt(_rules.line(25, 5, 4, "ab2", 4, "rng"), 8) == 0
