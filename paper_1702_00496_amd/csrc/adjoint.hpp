// Discrete adjoint of the AT step: parameters and launchers shared by
// adjoint.hip and the host front end in atfd.cpp.
#pragma once

#include "atfd_internal.hpp"

namespace atfd {

constexpr int kAdjBlocks = 1024;   // fixed grid of the lambda kernel: its alpha partials

// One stage of the reversed step n (see adjoint.hip): mu = m0 y0 + m1 y1,
// out = b0 x0 + b1 x1 + (transposed stage) + drained adjoint ring.
struct AdjParams {
  StepParams sp;                   // the forward problem (taps, delays, ring layout)
  int64_t n;                       // the step being reversed (n -> n + 1)
  int64_t npts;
  int burgers;                     // Burgers right-hand side (taps depend on the stage field)
  const void* y0;
  const void* y1;
  double m0, m1;
  const void* x0;
  const void* x1;
  double b0, b1;
  void* out;                       // the stage's adjoint field
  const void* levels;              // stored levels of the stage field from seg_start, npts apart
  int64_t seg_start;
  const void* fring;               // that field's ring of the segment: fslots slots, level l in l mod fslots
  int fslots, fslot;               // (fslot = n mod fslots)
  int64_t nsteps;                  // steps of the whole run
  void* hbuf;                      // forward halo values of this stage [pe][face strips]
  int64_t pfo[6];                  // offset of face f's strip inside one PE's pe_block values
  void* aring;                     // adjoint ring of the stage field, anslots slots (3-D kernel: the g ring)
  int anslots, gslot;              // (gslot = n mod anslots)
  double* partial;                 // [adj_partials] alpha-gradient partial sums
  double wt[kMaxL][kMaxT];         // level weights c_m(k) of every delay k < L (host-computed)
};

// The 3-D stage kernel (adjoint3d.hpp): PEs whose plane takes at most 1024
// threads of two points each, and whose x / y frame one item each.
inline int adj3d_threads(const StepParams& p) {
  const int64_t vec = static_cast<int64_t>((p.bx + 1) / 2) * p.by, items = 2 * static_cast<int64_t>(p.s) * (p.bx + p.by);
  int64_t t = vec > items ? vec : items;
  if (t < 192) t = 192;   // the face set-up's threads
  return static_cast<int>((t + 63) / 64 * 64);
}
inline size_t adj3d_lds(const StepParams& p, int w, bool m1) {
  const size_t S = p.s, W = (p.bx + 4 + S + 2) & ~size_t(1), H = p.by + 2 * S, nh = 2 * S * (p.bx + p.by);
  return 2 * nh * sizeof(double) + 2 * W * H * (m1 ? sizeof(double) : w) + 2 * W * H * w + S * p.bx * p.by * w;
}
inline bool adj3d_applies(const StepParams& p, bool f64) {
  // (with the wider planes of a second mu term; 8 KB for the static part)
  return p.ndim == 3 && adj3d_threads(p) <= 1024 && adj3d_lds(p, f64 ? 8 : 4, true) <= kLdsLimit - 8 * 1024;
}
// The 1-D / 2-D stage kernel (adjoint2d.hpp): the PE's plane in LDS, two points
// and at most two pairs of them ahead per thread, at least the face set-up's
// 192 threads.
inline int adj2d_threads(const StepParams& p) {
  const int64_t vec = static_cast<int64_t>((p.bx + 1) / 2) * (p.ndim == 2 ? p.by : 1);
  int64_t t = (vec + 63) / 64 * 64;
  if (t < 192) t = 192;
  return static_cast<int>(t < 1024 ? t : 1024);
}
inline size_t adj2d_lds(const StepParams& p, int w, bool m1) {
  const size_t S = p.s, by = p.ndim == 2 ? p.by : 1, W = (p.bx + 4 + S + 2) & ~size_t(1), H = by + (p.ndim == 2 ? 2 * S : 0),
               nh = 2 * S * by + (p.ndim == 2 ? 2 * S * p.bx : 0);
  return nh * sizeof(double) + W * H * ((m1 ? sizeof(double) : w) + w);
}
inline bool adj2d_applies(const StepParams& p, bool f64) {
  return p.ndim <= 2 && adj2d_lds(p, f64 ? 8 : 4, true) <= kLdsLimit - 8 * 1024;
}
inline bool adj_gather(const StepParams& p, bool f64) { return adj2d_applies(p, f64) || adj3d_applies(p, f64); }
hipError_t launch_adj1d_f32(const AdjParams& q, hipStream_t st);
hipError_t launch_adj1d_f64(const AdjParams& q, hipStream_t st);
hipError_t launch_adj2d_f32(const AdjParams& q, hipStream_t st);
hipError_t launch_adj2d_f64(const AdjParams& q, hipStream_t st);
hipError_t launch_adj3d_f32(const AdjParams& q, hipStream_t st);
hipError_t launch_adj3d_f64(const AdjParams& q, hipStream_t st);

// Copy levels lo .. lo + count - 1 between two rings of p's layout: level l
// from slot l mod ns of src to slot l mod nd of dst.
hipError_t launch_ring_levels(const StepParams& p, bool f64, const void* src, int ns, void* dst, int nd, int64_t lo,
                              int64_t count, hipStream_t st);

int adj_blocks(int64_t npts);
// alpha-gradient partial sums the stage kernels write (>= kAdjBlocks; one per
// PE for the PE-tiled kernel)
int adj_partials(const StepParams& p);
hipError_t launch_adj_step(const AdjParams& q, bool f64, hipStream_t st);
hipError_t launch_adj_sum(const double* partial, int count, double* out, hipStream_t st);

}  // namespace atfd
