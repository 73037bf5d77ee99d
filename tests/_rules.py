"""The library's dispatch rules on the host: the inline functions of its headers
in a small library of their own, compiled without device code."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "adjoint.hpp"
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
