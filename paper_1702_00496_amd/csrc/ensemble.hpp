// Delay ensembles: descriptors and launchers shared by ensemble.hip and the
// host front end ensemble_api.cpp.
#pragma once

#include "line.hpp"

namespace atfd {

// One member of the ensemble: a periodic 1-D advection-diffusion problem.
struct EnsMember : Line {
  int64_t off;                     // first point in the packed fields
  int64_t ring_off;                // first value of its ring in the packed ring
  int64_t hoff;                    // first value of its halo values in the packed halo buffer
  int vec;                         // 4-point vector sweep (b % 4 == 0 and off % 4 == 0)
  LinePlan plan;                   // on its compute unit (pt = 0: streamed), for the schedule in force
  double length, c, alpha;         // for the exact solution
};

// Microseconds of a run of nsteps steps on the member's compute unit, kept there
// (beyond kEnsKeptStart) and streamed. A kept member's whole state passes its
// compute unit twice whatever the steps, so short runs are streamed. Fitted to
// runs of 1 to 64 steps of 1024 to 65536 points, orders 2 and 4; the choice took
// at most 20 % longer than the better (one of 280 runs 35 %, at 3 steps). 512 members of 8192 points (two a compute
// unit), fourth order, FP64, kept / streamed: 1 step 81 / 33, 3 steps 88 / 77, 4
// steps 91 / 98; 64 of 4096, second order, FP32: 1 step 15 / 17.
constexpr double kEnsKeptStart = 6.0;
struct EnsTimes {
  double kept, streamed;
};
inline EnsTimes ens_times(const EnsMember& m, int w, int64_t nsteps) {
  const double steps = static_cast<double>(nsteps);
  const double fields = static_cast<double>(m.n) * w * (m.integrator == AT_AB2 ? 4 : 2);   // read and written a step
  const double ring = static_cast<double>(line_lds_ring(m.s, m.npe, m.nslots, m.integrator, w));
  EnsTimes t;
  t.streamed = steps * (2.45 + fields / 25000.0);
  t.kept = m.plan.pt ? (fields + 2.0 * ring) / (w == 4 ? 17000.0 : 13000.0) +
                           steps * (0.5 + fields / 210000.0 * (w == 8 && m.plan.fglob ? 4 : 1))
                     : t.streamed;
  return t;
}

struct EnsParams {
  const EnsMember* mem;            // [count]
  const int* bin_start;            // [nbins + 1] ranges of `order`
  const int* order;                // member ids, grouped by workgroup
  void* u[2];                      // packed fields, u^n in u[n & 1]
  void* f;                         // packed f^{n-1} (AB2 members)
  void* ring;                      // packed rings [member][slot][pe][face][s]
  void* hbuf;                      // packed halo values of the current step [member][pe][side][s]
  int64_t* counter;                // [0] = step n, [1] = finished workgroups
  int64_t nsteps;                  // steps of this launch
  int64_t lds;                     // dynamic LDS bytes of a workgroup
};

struct EnsNormParams {
  const EnsMember* mem;
  const void* u;                   // packed current fields
  const double* ref;               // packed reference (nmodes == 0)
  int64_t nstep;
  int nmodes;
  int kap[kMaxModes];
  double amp[kMaxModes];
  const double* phase;             // [count][nmodes], device
  double* out;                     // [count][4]: sum|E|, sum E^2, max|E|, non-finite count
};

struct EnsStatsParams {
  const EnsMember* mem;
  const double* sums;              // [count][4] from the norms kernel (sum E^2 at [1])
  const double* edges;             // [nbins + 1] ascending dx bin edges
  int count, nbins;
  double* out;                     // [3 groups][nbins][4]: count, mean dx, mean rms, unbiased variance
};

hipError_t launch_ens_stats(const EnsStatsParams& p, hipStream_t st);
// `small`: every member is kept on its compute unit with at most ens_small_pt
// points per thread (the lighter kernel, two 1024-thread workgroups per CU).
// `streamed`: no member is kept.
inline __host__ __device__ constexpr int ens_small_pt(bool f64) { return f64 ? 4 : 8; }
constexpr int kEnsMaxPt = 64;
hipError_t launch_ens_steps(const EnsParams& p, bool f64, bool small, bool streamed, int nbins, int threads,
                            hipStream_t st);
// Static LDS of a workgroup of the steps kernel.
int64_t ens_static_lds(bool small);
hipError_t launch_ens_publish_level0(const EnsParams& p, bool f64, int count, hipStream_t st);
hipError_t launch_ens_norms(const EnsNormParams& p, bool f64, int count, hipStream_t st);

}  // namespace atfd
