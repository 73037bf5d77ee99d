// Small 1-D contexts (time-expanded schemes and the synchronous arm): all
// steps of an at_step call in one launch of one workgroup that keeps the whole
// line on its compute unit (line.hpp).
//
// A step of the per-step sweep costs a launch and its memory round trips,
// about 6 us whatever the size; here it is a chain of LDS reads and one
// barrier (Heun: two). 256 points in 8 PEs, second order, Euler, FP64: 5.9 -> 0.5
// us a step; 252 points in 6 PEs, fourth-order Burgers, AB2, FP64: 6.8 -> 0.8 us.
// (Compiled for 1024 threads at any size: the sixth-order FP64 forms spill.)

#include "line.hpp"

namespace atfd {
namespace {

template <typename Real, int S, int PT, int KIND, int EQ>
__global__ __launch_bounds__(kMaxSweepThreads) void line_steps_kernel(LineSteps q) {
  extern __shared__ __align__(16) unsigned char line_smem[];
  const int64_t n0 = q.counter[0];
  LineBufs<Real> B;
  B.u_in = static_cast<const Real*>(q.ubuf[n0 & 1]);
  B.u_out = static_cast<Real*>(q.ubuf[(n0 + q.nsteps) & 1]);
  B.f0 = static_cast<Real*>(q.fbuf[0]);
  B.f1 = static_cast<Real*>(q.fbuf[1]);
  B.ustar = static_cast<Real*>(q.ustar);
  B.ring = static_cast<Real*>(q.ring);
  B.sring = static_cast<Real*>(q.sring);
  B.host = q.host;
  if constexpr (sizeof(Real) == 8) {
    B.lap = q.lap;
    B.grd = q.grd;
  } else {
    B.lap = q.lapf;
    B.grd = q.grdf;
  }
  line_run<Real, S, PT, S + 1, KIND, EQ, false, false, true>(q.line, q.plan, B, n0, q.nsteps, line_smem);
  // (every thread has read n0: line_run ends with a barrier)
  if (threadIdx.x == 0) q.counter[0] = n0 + q.nsteps;
}

template <typename Real, int S, int PT, int KIND>
void launch_eq(const LineSteps& q, int threads, size_t lds, hipStream_t st) {
  if (q.equation == AT_ADVDIFF)
    hipLaunchKernelGGL((line_steps_kernel<Real, S, PT, KIND, AT_ADVDIFF>), dim3(1), dim3(threads), lds, st, q);
  else
    hipLaunchKernelGGL((line_steps_kernel<Real, S, PT, KIND, AT_BURGERS>), dim3(1), dim3(threads), lds, st, q);
}

template <typename Real, int S, int PT>
hipError_t launch_kind(const LineSteps& q, int threads, size_t lds, hipStream_t st) {
  switch (q.line.integrator) {
    case AT_EULER: launch_eq<Real, S, PT, AT_EULER>(q, threads, lds, st); break;
    case AT_AB2: launch_eq<Real, S, PT, AT_AB2>(q, threads, lds, st); break;
    case AT_AB3: launch_eq<Real, S, PT, AT_AB3>(q, threads, lds, st); break;
    case AT_RK2: launch_eq<Real, S, PT, AT_RK2>(q, threads, lds, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename Real, int S>
hipError_t launch_pt(const LineSteps& q, int threads, size_t lds, hipStream_t st) {
  return q.plan.pt == 4 ? launch_kind<Real, S, 4>(q, threads, lds, st)
       : q.plan.pt == 8 ? launch_kind<Real, S, 8>(q, threads, lds, st)
                        : hipErrorInvalidValue;
}

template <typename Real>
hipError_t launch_s(const LineSteps& q, int threads, size_t lds, hipStream_t st) {
  switch (q.line.s) {
    case 1: return launch_pt<Real, 1>(q, threads, lds, st);
    case 2: return launch_pt<Real, 2>(q, threads, lds, st);
    case 3: return launch_pt<Real, 3>(q, threads, lds, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_line_steps(const LineSteps& q, bool f64, hipStream_t st) {
  const Line& M = q.line;
  const int w = f64 ? 8 : 4;
  const int64_t chunks = static_cast<int64_t>(q.plan.c) * M.npe;
  if (q.plan.pt < 4 || q.plan.glob || chunks < 1 || chunks > kMaxSweepThreads ||
      static_cast<int64_t>(q.plan.c) * q.plan.pt - q.plan.nshort != M.b)
    return hipErrorInvalidValue;
  const int64_t lds = line_lds_base(M.s, static_cast<int>(chunks), M.integrator, w) +
                      line_lds_ring(M.s, M.npe, M.nslots, M.integrator, w);
  if (lds > static_cast<int64_t>(kLdsLimit)) return hipErrorInvalidValue;
  const int threads = static_cast<int>((chunks + 63) / 64 * 64);
  return f64 ? launch_s<double>(q, threads, static_cast<size_t>(lds), st)
             : launch_s<float>(q, threads, static_cast<size_t>(lds), st);
}

}  // namespace atfd
