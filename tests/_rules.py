"""The library's dispatch rules on the host: the inline functions of its headers
in a small library of their own, compiled without device code."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "adjoint.hpp"
#include "ensemble.hpp"
#include "line.hpp"
using namespace atfd;
// 0: strip and stage kernels of adjoint.hip, 2: 1-D / 2-D stage kernel, 3: 3-D stage kernel
extern "C" int adjoint_kernel(int ndim, const int* b, const int* pe, int s, int integrator, int equation, int f64) {
  StepParams p{};
  p.ndim = ndim;
  p.bx = b[0]; p.by = b[1]; p.bz = b[2];
  p.px = pe[0]; p.py = pe[1]; p.pz = pe[2];
  p.npe = pe[0] * pe[1] * pe[2];
  p.s = s;
  p.integrator = integrator;
  p.equation = equation;
  for (int a = 0; a < ndim; ++a) p.pe_block += 2LL * s * b[0] * b[1] * b[2] / b[a];
  return adj3d_applies(p, f64 != 0) ? 3 : adj2d_applies(p, f64 != 0) ? 2 : 0;
}
// {n, pe, s, T, L, integrator, mode} of a line
static Line line(const int* v) {
  Line M{};
  M.n = v[0]; M.npe = v[1]; M.b = v[0] / v[1]; M.s = v[2]; M.T = v[3]; M.L = v[4];
  M.integrator = v[5]; M.mode = v[6];
  M.nslots = M.mode == AT_SYNC ? 0 : M.L + M.T;
  return M;
}
// {pt, c, nshort, glob, fglob}
extern "C" void plan(const int* v, int w, int threads, long long lds, int max_pt, int share, int* out) {
  const LinePlan p = line_plan(line(v), w, threads, lds, max_pt, share);
  out[0] = p.pt; out[1] = p.c; out[2] = p.nshort; out[3] = p.glob; out[4] = p.fglob;
}
// the plan of an ensemble member on one workgroup of `threads` threads a compute unit
extern "C" void member_plan(const int* v, int w, int threads, int* out) {
  // (24 descriptors of a batch and their indices, rounded up)
  const long long fixed = (AT_ENS_BATCH * static_cast<long long>(sizeof(EnsMember) + sizeof(int)) + 255) / 256 * 256;
  plan(v, w, threads, static_cast<long long>(kLdsLimit) - fixed, kEnsMaxPt, 1, out);
}
// a context: its plan, 0 where it is stepped launch by launch
extern "C" int context_pt(const int* v, int w) {
  return line_plan(line(v), w, kMaxSweepThreads, static_cast<int64_t>(kLdsLimit), kLineMaxPt, 1).pt;
}
// microseconds of `count` such members on one compute unit: {kept, streamed}
extern "C" void ens(const int* v, int w, int count, long long nsteps, double* out) {
  EnsMember m{};
  static_cast<Line&>(m) = line(v);
  m.plan = line_plan(m, w, 1024, static_cast<int64_t>(kLdsLimit) - 16384, kEnsMaxPt, 1);
  const EnsTimes t = ens_times(m, w, nsteps);
  out[0] = kEnsKeptStart + count * t.kept;
  out[1] = count * t.streamed;
}
extern "C" int pays(const int* v, int w, long long nsteps) { return line_pays(line(v), w, nsteps); }
"""


def build(tmp):
    from paper_1702_00496_amd import build as B
    src, out = os.path.join(tmp, "rules.hip"), os.path.join(tmp, "rules.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    cmd = [B.hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", B.CSRC, "-I", B.INCLUDE,
           src, "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode:
        pytest.fail(res.stderr[-2000:])
    return ctypes.CDLL(out)


def three(v):
    v = tuple(v) + (1,) * (3 - len(v))
    return (ctypes.c_int * 3)(*v)


def adjoint_kernel(lib, n, pe, order, integrator, equation, precision):
    b = [x // y for x, y in zip(n, pe)]
    return lib.adjoint_kernel(len(n), three(b), three(pe), order // 2, {"euler": 0, "ab2": 1, "rk2": 3}[integrator],
                              {"advdiff": 0, "burgers": 1}[equation], int(precision == "f64"))


INTEGRATORS = {"euler": 0, "ab2": 1, "ab3": 2, "rk2": 3}
MODES = {"rng": 0, "zero": 1, "host": 2, "sync": 3}


def line(n, pe, order, integrator, L, mode, T=0):
    s = order // 2
    return (ctypes.c_int * 7)(n, pe, s, 1 if mode == "sync" else T or s + 1, 1 if mode == "sync" else L,
                              INTEGRATORS[integrator], MODES[mode])


def width(precision):
    return 8 if precision == "f64" else 4
