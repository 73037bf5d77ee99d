// The arithmetic of a 1-D step, written with explicit fused multiply-adds and
// shared by everything that advances a 1-D problem of the time-expanded schemes:
// the line kept on a compute unit (line.hpp), the streamed ensemble member
// (ensemble.hip) and the sweep (step_sweep.hpp). They round alike, so that the
// path a launch takes, a schedule and a split of a run change no bit.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace atfd {

__device__ inline float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }

// One level of the AT combination, in double (a weight of zero drops it).
template <typename Real>
__device__ inline double add_level(double acc, double w, Real v) {
  return w != 0.0 ? fmadd(w, static_cast<double>(v), acc) : acc;
}

// acc + the taps at -o and +o of the differences xm, xp to the centre.
template <typename Real>
__device__ inline Real add_pair(Real acc, Real tm, Real xm, Real tp, Real xp) {
  return fmadd(tp, xp, fmadd(tm, xm, acc));
}
// Burgers: alpha (Laplacian l) - u0 (gradient g).
template <typename Real>
__device__ inline Real burgers_rhs(Real u0, Real l, Real g) {
  return fmadd(-u0, g, l);
}

template <typename Real>
__device__ inline Real euler_update(Real u0, Real dt, Real f) {
  return fmadd(dt, f, u0);
}
// u + dt (b1 f + b2 f^{n-1}): AB2 (b1 = 3/2, b2 = -1/2), or Euler with b2 = 0
// (AB2's first step: b1 = 1 and fo must be finite).
template <typename Real>
__device__ inline Real ab2_update(Real u0, Real dt, Real b1, Real f, Real b2, Real fo) {
  return fmadd(dt, fmadd(b1, f, b2 * fo), u0);
}
// AB3 (23, -16, 5)/12 at step n; Euler at n = 0, AB2 at n = 1 (f^{n-1} and
// f^{n-2} must be finite where they do not exist yet).
template <typename Real>
struct Ab3 {
  Real c0, c1, c2;
  __device__ explicit Ab3(int64_t n)
      : c0(n == 0 ? Real(1) : n == 1 ? Real(1.5) : Real(23.0 / 12.0)),
        c1(n == 0 ? Real(0) : n == 1 ? Real(-0.5) : Real(-16.0 / 12.0)), c2(n >= 2 ? Real(5.0 / 12.0) : Real(0)) {}
};
template <typename Real>
__device__ inline Real ab3_update(Real u0, Real dt, const Ab3<Real>& c, Real f, Real f1, Real f2) {
  return fmadd(dt, fmadd(c.c2, f2, fmadd(c.c1, f1, c.c0 * f)), u0);
}
// Heun's second stage: (u^n + u*) / 2 + dt / 2 f(u*).
template <typename Real>
__device__ inline Real heun_update(Real un, Real us, Real dt, Real f) {
  return fmadd(Real(0.5) * dt, f, Real(0.5) * (un + us));
}

}  // namespace atfd
