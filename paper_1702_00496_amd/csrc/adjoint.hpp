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
  void* aring;                     // anslots slots: the stage field's g ring (gathering kernels), or its adjoint
                                   // ring, in double (strip and stage kernels)
  int anslots, gslot;              // (gslot = n mod anslots)
  double* partial;                 // [adj_partials] alpha-gradient partial sums
  double wt[kMaxL][kMaxT];         // level weights c_m(k) of every delay k < L (host-computed)
};

// The 3-D stage kernel (adjoint3d.hpp) takes PEs whose plane has at most 1024
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
inline bool adj3d_fits(const StepParams& p, bool f64) {
  // (with the wider planes of a second mu term; 8 KB for the static part)
  return p.ndim == 3 && adj3d_threads(p) <= 1024 && adj3d_lds(p, f64 ? 8 : 4, true) <= kLdsLimit - 8 * 1024;
}
// Whether it is the faster one. It walks a PE's planes one after the other in
// one workgroup: its time follows the planes, whatever the number of PEs, until
// they fill the chip. The strip and stage kernels of adjoint.hip spread the
// points over the chip: their time follows the points and the strip values.
// Microseconds a stage, measured alone over 18 shapes, orders 2 to 6, both
// equations, one and two mu terms, FP32 and FP64 (432 cases; the choice made
// here took at most 12 % longer than the better of the two):
//   24 x 24 x 96, 2 x 2 x 1 PEs, order 4, FP32 / FP64: 182 / 191 here, 30 / 31 there;
//   32^3, 2^3 PEs, order 6 Burgers: 108 / 234, 41 / 41; 8 x 8 x 4 PEs: 128 / 363, 872 / 1010;
//   64 x 32 x 32 (1024 threads, whose 128 registers spill), order 4, 2^3 PEs:
//   227 / 432, 43 / 46; 4 x 8 x 8 PEs: 380 / 752, 1061 / 1282;
//   6^3, 16^3 PEs, order 4: 166 / 172, 112 / 128.
inline bool adj3d_pays(const StepParams& p, bool f64) {
  constexpr double kPlane[2][3] = {{1.45, 1.85, 2.6}, {1.5, 2.0, 4.5}};        // up to 512 threads: FP32, FP64
  constexpr double kPlaneWide[2][3] = {{2.6, 7.0, 13.5}, {5.5, 13.2, 13.2}};   // 1024 threads
  constexpr double kPoint[2][3] = {{23.0, 53.0, 78.0}, {26.0, 66.0, 95.0}};    // a million points
  constexpr double kStrip = 18.0;                                             // a million strip values
  const int i = f64 ? 1 : 0, j = p.s - 1, threads = adj3d_threads(p);
  const bool wide = threads > 512, burgers = p.equation == AT_BURGERS;
  // (a second mu term, AB2's, costs the wide FP32 forms most of their spills)
  const double plane = wide ? kPlaneWide[i][j] * (!f64 && p.integrator != AT_AB2 ? 0.6 : 1.0)
                     : f64 && j == 2 && burgers ? 7.0 : kPlane[i][j];
  // eight waves a compute unit (256 registers), 256 compute units
  const int64_t at_once = 256 * (wide ? 1 : 512 / threads);
  const double rounds = static_cast<double>((p.npe + at_once - 1) / at_once);
  const double here = rounds * (8.0 + 3.0 * j + plane * p.bz);
  const double pts = 1e-6 * p.npe * p.bx * p.by * p.bz, strips = 1e-6 * p.npe * static_cast<double>(p.pe_block);
  const double there = 15.0 + 4.0 * j + pts * kPoint[i][j] * (burgers ? 1.17 : 1.0) + strips * kStrip;
  return here <= there;
}
inline bool adj3d_applies(const StepParams& p, bool f64) { return adj3d_fits(p, f64) && adj3d_pays(p, f64); }
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
