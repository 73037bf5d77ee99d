// A periodic 1-D problem kept on one compute unit for all steps of a launch
// (Sec. 2, Sec. 4.1): the members of a delay ensemble and the small 1-D
// contexts. One workgroup owns the whole line. Its points live in registers,
// PT consecutive ones of one PE per thread (a chunk); chunks exchange their
// edge values, and PEs read their neighbours' past levels, through LDS, so a
// step needs one workgroup barrier (Heun: two) and no memory traffic.
//
// What bounds it: for short lines the chain of a step (edge reads from LDS, the
// stencil, the publish, the barrier), for long ones the vector arithmetic of
// one compute unit (about 10 instructions a point for fourth-order AB2). Off
// the chain: the level combinations are made a step ahead (all their levels
// are published by then; a face without a delay takes its neighbour's current
// edge), and the delays, which do not depend on the field, are drawn for a
// batch of steps at a time by all threads. Microseconds a step, FP32, order 2
// / fourth-order AB2 with L = 2: 1024 points 0.51 / 0.76, 8192 0.85 / 1.26,
// 32768 1.53 / 3.17, 65536 2.84 / 6.58 (streamed through the caches: 65536
// points, fourth order, about 30); a sweep per step of a 1-D context 5 to 6.
#pragma once

#include "atfd_internal.hpp"
#include "update.hpp"

namespace atfd {

// One 1-D problem (uniform over its workgroup).
struct Line {
  int64_t n;                       // points
  int b, npe, s, T, L, nslots;     // PE edge, PEs, half-width, levels, max delay, ring slots
  int integrator, mode;            // AT_EULER .. AT_RK2; AT_DELAY_* | AT_SYNC
  uint64_t key;                    // generator key
  uint64_t thr[kMaxL];             // delay bin thresholds (ascending)
  double wt[kMaxL][kMaxT];         // level weights c_m(k) for every delay k < L
  double dt;
  double kad[2 * kMaxS + 1];       // alpha c2/dx^2 - c c1/dx per tap o = -s..s
  float kadf[2 * kMaxS + 1];
};

// How a line is laid over the threads of a workgroup: PT points per chunk, C
// chunks per PE, of which the last `nshort` hold PT - 1 points. glob: the
// ring stays in device memory (it does not fit LDS), and with fglob the AB2
// history too (it does not fit the registers beside PT points of u).
struct LinePlan {
  int pt, c, nshort, glob, fglob;
};

// Delays drawn ahead: two halves of kLineDelays bytes, one byte per face and
// step, used alternately. A workgroup has a thread per PE at least, so a half
// always covers two steps.
constexpr int kLineDelays = 4096;
constexpr int kLineMaxThreads = 1024;
static_assert(kLineDelays >= 2 * (2 * kLineMaxThreads), "line_run's batches are of two steps or more");

inline __host__ __device__ int line_batch(int faces) {
  const int r = kLineDelays / faces;
  return r < 1 ? 1 : r > 64 ? 64 : r;
}

// LDS bytes of a line's run without its ring, and of its ring (one level ring;
// Heun keeps a second one and a second set of edge values).
inline __host__ __device__ int64_t line_lds_base(int s, int chunks, int integrator, int w) {
  const int64_t edges = static_cast<int64_t>(4) * s * chunks * w * (integrator == AT_RK2 ? 2 : 1);
  return kMaxL * kMaxT * 8 + 2 * kLineDelays + (edges + 15) / 16 * 16;
}
inline __host__ __device__ int64_t line_lds_ring(int s, int npe, int nslots, int integrator, int w) {
  return static_cast<int64_t>(2) * s * npe * nslots * w * (integrator == AT_RK2 ? 2 : 1);
}

// The plan of a line on `threads` threads and `lds` bytes, with at most
// `max_pt` points per thread, where `share` such workgroups are on a compute
// unit; pt = 0 if there is none. A step costs a wave about 180 instructions
// and 12 a point, and the waves of a SIMD take turns: the PT with the smallest
// product of waves per SIMD and instructions per wave is taken (4096 points,
// fourth-order AB2, FP32: 1.63 us a step with 4 points per thread, 1.00 with 16).
// Registers hold u and, for AB2, f: 32 FP32 (16 FP64) points of both or twice as
// many of u alone, out of the 128 registers a thread of a 1024-thread workgroup
// has; one size above that AB2 keeps f in device memory (whole chunks only: it is
// stored chunk-transposed), which costs about twice as much.
inline __host__ __device__ LinePlan line_plan(const Line& M, int w, int threads, int64_t lds, int max_pt, int share) {
  LinePlan best{0, 0, 0, 0, 0};
  // (the kernels combine the schemes' own level count)
  if (M.mode != AT_SYNC && M.T != M.s + 1) return best;
  if (threads > kLineMaxThreads || M.b < 2 * M.s) return best;
  const int reg_pt = w == 4 ? 64 : 32;   // u alone
  int64_t best_cost = 0;
  for (int pt = 4; pt <= max_pt && pt <= reg_pt; pt *= 2) {
    const int c = (M.b + pt - 1) / pt, ns = c * pt - M.b;
    if (ns > c || pt - (ns ? 1 : 0) < M.s) continue;
    const int64_t chunks = static_cast<int64_t>(c) * M.npe;
    if (chunks > threads) continue;
    const int fglob = M.integrator == AT_AB2 && pt == reg_pt ? 1 : 0;
    if (fglob && ns) continue;
    const int64_t base = line_lds_base(M.s, static_cast<int>(chunks), M.integrator, w);
    const int64_t ring = line_lds_ring(M.s, M.npe, M.nslots, M.integrator, w);
    int glob = 0;
    if (base + ring > lds) {
      // the ring in device memory: only for long chunks, whose arithmetic
      // covers the reads
      if (base > lds || pt < 16) continue;
      glob = 1;
    }
    const int64_t cost = ((chunks * share + 255) / 256) * (180 + 12 * pt) * (fglob ? 2 : 1);
    if (best.pt && cost >= best_cost) continue;
    best = LinePlan{pt, c, ns, glob, fglob};
    best_cost = cost;
  }
  return best;
}

// A launch that advances a whole 1-D context nsteps steps (line.hip).
constexpr int kLineMaxPt = 8;      // points per thread of such a launch
// Steps of one launch: 8 to 80 ms, so that a long call leaves the device gaps to
// take other work in (a launch costs 4 to 13 us).
constexpr int64_t kLineMaxSteps = 1 << 14;
struct LineSteps {
  Line line;
  LinePlan plan;
  int equation;
  double lap[2 * kMaxS + 1], grd[2 * kMaxS + 1];   // Burgers taps alpha c2, c1
  float lapf[2 * kMaxS + 1], grdf[2 * kMaxS + 1];
  void* ubuf[2];
  void* fbuf[2];
  void* ustar;
  void* ring;
  void* sring;
  const int8_t* host;
  int64_t* counter;
  int64_t nsteps;
};
hipError_t launch_line_steps(const LineSteps& q, bool f64, hipStream_t st);

// Whether a call of nsteps steps of a context with such a plan takes that
// launch or a sweep per step (they round alike: update.hpp). The launch reads
// and writes the whole state through one compute unit whatever the steps, so a
// call of one or two steps of a large state is faster as sweeps. Microseconds
// fitted to calls of 1 to 3 steps of 256 to 8192 points, within 10 % of the
// better: 8192 points, fourth-order AB2, L = 8, FP64: 1 step 13.1 (sweep 6.3), 2
// steps 15.1 (11.6), 3 steps 17.0 (16.9); 1024 points 5.5 (6.2).
inline bool line_pays(const Line& M, int w, int64_t nsteps) {
  const int fields[4] = {2, 4, 6, 3};   // read and written: Euler, AB2, AB3, Heun
  const int stages = M.integrator == AT_RK2 ? 2 : 1;
  const double io = static_cast<double>(M.n) * w * fields[M.integrator] +
                    2.0 * static_cast<double>(line_lds_ring(M.s, M.npe, M.nslots, M.integrator, w));
  // (the sixth-order FP64 forms spill)
  const double stage = w == 8 && M.s == 3 ? 1.5 + 5.5e-4 * static_cast<double>(M.n)
                                          : 0.25 + 7.5e-5 * static_cast<double>(M.n) * M.s;
  const double steps = static_cast<double>(nsteps) * stages;
  return 3.7 + io / 45000.0 + steps * stage <= 0.6 + 5.4 * steps;
}

// Device memory of one line's run: the fields at its first and last step, the
// history (f0; AB3 also f1, by step parity), the predictor (Heun), the rings,
// a host delay table [step][pe][side].
template <typename Real>
struct LineBufs {
  const Real* u_in;
  Real* u_out;
  Real* f0;
  Real* f1;
  Real* ustar;
  Real* ring;
  Real* sring;
  const int8_t* host;
  const Real* lap;   // Burgers taps (alpha c2, c1), else null
  const Real* grd;
};

// All steps n0 .. n0 + nsteps - 1 of one line.
//  FACE_MAJOR: a ring slot holds [face][pe][depth] (a context's ring), else
//  [pe][face][depth] (a member's);
//  TT: levels of a combination, S + 1 (the synchronous arm combines none);
//  KIND: integrator; EQ: equation; GR: the ring stays in device memory;
//  FG: the AB2 history too, chunk-transposed in the u_out buffer during the
//  run ([4-value group][chunk], so that a wave's accesses are contiguous).
// Long chunks are walked four points at a time (a scheduling barrier between
// the groups), which keeps the values in flight inside the registers.
template <typename Real, int S, int PT, int TT, int KIND, int EQ, bool GR, bool FG, bool FACE_MAJOR>
__device__ __forceinline__ void line_run(const Line& Mref, const LinePlan& pl, const LineBufs<Real>& B, int64_t n0,
                                         int64_t nsteps, unsigned char* smem) {
  constexpr bool kRk2 = KIND == AT_RK2;
  // long chunks: 128 bytes of points and more; the point before which one
  // issues the reads of the next step's halos (FP64: after the last)
  constexpr bool kLong = PT * sizeof(Real) >= 128;
  constexpr int kLate = !kLong ? -1 : sizeof(Real) == 4 ? PT - 16 : PT;
  constexpr bool kAb = KIND == AT_AB2 || KIND == AT_AB3;
  static_assert(!FG || KIND == AT_AB2, "only the AB2 history is kept in device memory");
  const int tid = threadIdx.x, nt = blockDim.x;
  const int b = uniform(Mref.b), npe = uniform(Mref.npe), L = uniform(Mref.L);
  const int nslots = uniform(Mref.nslots), mode = uniform(Mref.mode);
  const int C = uniform(pl.c), nshort = uniform(pl.nshort);
  const int nch = C * npe, faces = 2 * npe;
  const bool sync = mode == AT_SYNC;
  const Real dt = uniform(static_cast<Real>(Mref.dt));
  // LDS: level weights, the delays drawn ahead, edge values, the ring
  double* s_wt = reinterpret_cast<double*>(smem);
  int8_t* s_k = reinterpret_cast<int8_t*>(smem + kMaxL * kMaxT * 8);
  Real* s_e = reinterpret_cast<Real*>(smem + kMaxL * kMaxT * 8 + 2 * kLineDelays);
  const int eset = 2 * S * nch;                     // edge values of one level
  const int64_t ebytes = static_cast<int64_t>(4) * S * nch * sizeof(Real) * (kRk2 ? 2 : 1);
  Real* s_ring = reinterpret_cast<Real*>(smem + kMaxL * kMaxT * 8 + 2 * kLineDelays + (ebytes + 15) / 16 * 16);
  // ring values of one slot (the synchronous arm has no ring: its halo reads,
  // of which nothing is used, go to the edge values)
  const int rstride = sync ? 0 : faces * S;
  const int rtotal = rstride * nslots;
  Real* s_sring = s_ring + rtotal;
  Real* ring = sync ? s_e : GR ? B.ring : s_ring;
  Real* sring = sync ? s_e : GR ? B.sring : s_sring;

  Real kad[2 * S + 1], lap[2 * S + 1], grd[2 * S + 1];
#pragma unroll
  for (int o = 0; o <= 2 * S; ++o) {
    if constexpr (EQ == AT_ADVDIFF) {
      if constexpr (sizeof(Real) == 8) kad[o] = uniform(Mref.kad[o]);
      else kad[o] = uniform(Mref.kadf[o]);
    } else {
      lap[o] = uniform(B.lap[o]);
      grd[o] = uniform(B.grd[o]);
    }
  }

  // this thread's chunk
  const bool active = tid < nch;
  const int pe = active ? tid / C : 0, ci = active ? tid - pe * C : 0;
  const bool is_short = ci >= C - nshort;
  const int len = is_short ? PT - 1 : PT;
  const int off = pe * b + ci * PT - (is_short ? ci - (C - nshort) : 0);   // first point
  const bool hasL = ci == 0, hasR = ci == C - 1;
  const int tl = tid == 0 ? nch - 1 : tid - 1, tr = tid + 1 == nch ? 0 : tid + 1;   // neighbour chunks (periodic)
  const int ql = pe == 0 ? npe - 1 : pe - 1, qr = pe + 1 == npe ? 0 : pe + 1;       // neighbour PEs

  Real u[PT], us[kRk2 ? PT : 1], fa[(kAb && !FG) ? PT : 1], fb[KIND == AT_AB3 ? PT : 1];
  // (loads without a branch: idle threads read chunk 0, a short chunk its last
  // point twice)
  auto at = [&](int e) __attribute__((always_inline)) { return off + (e < PT - 1 ? e : len - 1); };
#pragma unroll
  for (int e = 0; e < PT; ++e) u[e] = B.u_in[at(e)];
  Real* fT = B.u_out;   // FG: transposed history, group g of 4 values at (g nch + chunk) 4
  if constexpr (FG) __syncthreads();   // u_out may be u_in: every chunk is loaded before it is written
  // group g of the transposed history: a uniform base and a 32-bit offset that
  // the loop may not hoist (one address a group would take 32 registers)
  constexpr int kAhead = 4;
  auto fT_at = [&](int g) __attribute__((always_inline)) {
    uint32_t o = static_cast<uint32_t>(tid) * 4u * sizeof(Real);
    asm volatile("" : "+v"(o));
    return reinterpret_cast<Real*>(reinterpret_cast<char*>(fT + static_cast<int64_t>(g) * nch * 4) + o);
  };
  auto get4 = [&](int g, Real (&v)[4]) __attribute__((always_inline)) {
    const Real* src = fT_at(g);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = src[j];
  };
  auto put4 = [&](int g, const Real (&v)[4]) __attribute__((always_inline)) {
    Real* dst = fT_at(g);
#pragma unroll
    for (int j = 0; j < 4; ++j) dst[j] = v[j];
  };
  if constexpr (kAb) {
    // f^{n-1} (and f^{n-2}); nothing is stored before the first step (second)
    const bool have = n0 > 0, have2 = KIND == AT_AB3 && n0 > 1;
    const Real* f1p = KIND == AT_AB3 ? (((n0 - 1) & 1) ? B.f1 : B.f0) : B.f0;
    const Real* f2p = KIND == AT_AB3 ? ((n0 & 1) ? B.f1 : B.f0) : nullptr;
    if constexpr (FG) {
      if (active)
#pragma unroll 4
        for (int g = 0; g < PT / 4; ++g) {
          Real v[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = have ? f1p[off + 4 * g + j] : Real(0);
          put4(g, v);
        }
    } else {
#pragma unroll
      for (int e = 0; e < PT; ++e) fa[e] = Real(0);
      if (have)
#pragma unroll
        for (int e = 0; e < PT; ++e) fa[e] = f1p[at(e)];
    }
    if constexpr (KIND == AT_AB3) {
#pragma unroll
      for (int e = 0; e < PT; ++e) fb[e] = Real(0);
      if (have2)
#pragma unroll
        for (int e = 0; e < PT; ++e) fb[e] = f2p[at(e)];
    }
  }
  for (int i = tid; i < kMaxL * kMaxT; i += nt) s_wt[i] = Mref.wt[i / kMaxT][i % kMaxT];
  if (!sync && !GR)
    for (int i = tid; i < rtotal; i += nt) {
      s_ring[i] = B.ring[i];
      if (kRk2) s_sring[i] = B.sring[i];
    }

  // Delays of `rows` steps from step n into half h (the draw of every delay
  // mode, clamped). The bins' thresholds ascend, so the bin is a count; bins
  // past L never count (u53 < 2^53). Threads step through (row, face) without
  // a division.
  uint64_t thr[kMaxL - 1];
#pragma unroll
  for (int j = 0; j < kMaxL - 1; ++j)
    thr[j] = static_cast<uint64_t>(uniform(static_cast<int64_t>(j < L - 1 ? Mref.thr[j] : ~0ull)));
  const uint64_t key = static_cast<uint64_t>(uniform(static_cast<int64_t>(Mref.key)));
  const int drow = uniform(nt / faces), dface = uniform(nt - nt / faces * faces);
  const int row0 = tid / faces, face0 = tid - row0 * faces;
  auto draw = [&](int64_t n, int rows, int h) __attribute__((always_inline)) {
    if (sync) return;
    int8_t* dst = s_k + h * kLineDelays;
    int row = row0, face = face0;
    for (int i = tid; row < rows; i += nt) {
      const int64_t nn = n + row;
      int k = 0;
      if (mode == AT_DELAY_RNG) {
        const uint64_t ctr = ((static_cast<uint64_t>(nn) << 32) | static_cast<uint32_t>(face)) + 1ull;
        const uint64_t u53 = mix64(key + ctr * kGolden) >> 11;
#pragma unroll
        for (int j = 0; j < kMaxL - 1; ++j) k += u53 >= thr[j] ? 1 : 0;
      } else if (mode == AT_DELAY_HOST) {
        k = B.host[nn * faces + face];
      }
      dst[i] = static_cast<int8_t>(clamp_startup(k, nn, TT));
      row += drow;
      face += dface;
      if (face >= faces) {
        face -= faces;
        ++row;
      }
    }
  };
  // strip of one face of a PE inside a ring slot
  auto strip_at = [&](int q, int face) __attribute__((always_inline)) {
    return FACE_MAJOR ? (face * npe + q) * S : (q * 2 + face) * S;
  };
  // first (last) S values of the chunk into edge set e: [side][depth][chunk]
  auto put_edges = [&](const Real* v, Real* e) __attribute__((always_inline)) {
#pragma unroll
    for (int d = 0; d < S; ++d) {
      e[d * nch + tid] = v[d];
      const Real full = v[PT - S + d], shrt = v[PT - S + d - 1];
      e[(S + d) * nch + tid] = is_short ? shrt : full;
    }
  };
  auto publish = [&](const Real* v, Real* R, int slot) __attribute__((always_inline)) {
    if (sync) return;
    if (hasL) {
      Real* dst = R + slot * rstride + strip_at(pe, 0);
#pragma unroll
      for (int d = 0; d < S; ++d) dst[d] = v[d];
    }
    if (hasR) {
      Real* dst = R + slot * rstride + strip_at(pe, 1);
#pragma unroll
      for (int d = 0; d < S; ++d) {
        const Real full = v[PT - S + d], shrt = v[PT - S + d - 1];
        dst[d] = is_short ? shrt : full;
      }
    }
  };
  // Delays of the chunk's PE at the step in row `row` of half `half`: low face
  // in bits 0-7, high face in bits 8-15 (the synchronous arm: 0).
  auto delays_at = [&](int row, int half) __attribute__((always_inline)) {
    if (sync) return 0;
    return static_cast<int>(*reinterpret_cast<const uint16_t*>(s_k + half * kLineDelays + row * faces + 2 * pe));
  };
  // The halo of one side for the step at ring position r (level l in slot r)
  // with delay k > 0: all its levels l - k - m are published by then. halo_raw
  // reads them, halo_sum combines them. k = 0 reads the slots of k = 1 and is
  // not used: such a face takes the neighbour's current edge.
  struct Raw {
    Real v[TT][S];
  };
  auto halo_raw = [&](int side, const Real* R, int r, int k, Raw& q) __attribute__((always_inline)) {
    const int kk = k > 0 ? k : 1;
    // the left neighbour's right strip (face 1), the right one's left strip
    const Real* strip = R + strip_at(side ? qr : ql, side ? 0 : 1);
    int o = r * rstride - static_cast<int>(__umul24(kk, rstride));   // slot r - kk
#pragma unroll
    for (int m = 0; m < TT; ++m) {
      const Real* lv = strip + (o < 0 ? o + rtotal : o);
      o -= rstride;
#pragma unroll
      for (int d = 0; d < S; ++d) q.v[m][d] = lv[d];
    }
  };
  auto halo_sum = [&](int k, const Raw& q, Real* h) __attribute__((always_inline)) {
    double acc[S];
#pragma unroll
    for (int d = 0; d < S; ++d) acc[d] = 0.0;
#pragma unroll
    for (int m = 0; m < TT; ++m) {
      const double w = s_wt[k * kMaxT + m];
#pragma unroll
      for (int d = 0; d < S; ++d) acc[d] = add_level(acc[d], w, q.v[m][d]);
    }
#pragma unroll
    for (int d = 0; d < S; ++d) h[d] = static_cast<Real>(acc[d]);
  };
  // The S values beyond each side of the chunk: the neighbour chunk's current
  // edge (from edge set e), or across a PE face with a delay the halo h.
  auto ghosts = [&](const Real* e, int k, const Real* hl, const Real* hr, Real* gl, Real* gr)
      __attribute__((always_inline)) {
    const bool ul = hasL && (k & 0xff) != 0, ur = hasR && (k >> 8) != 0;
#pragma unroll
    for (int d = 0; d < S; ++d) {
      const Real l = e[(S + d) * nch + tl], r = e[d * nch + tr];
      gl[d] = ul ? hl[d] : l;
      gr[d] = ur ? hr[d] : r;
    }
  };
  // right-hand side at every point of the chunk, given to put(e, u0, f)
  auto stencil = [&](const Real* v, const Real* gl, const Real* gr, auto put) __attribute__((always_inline)) {
    Real x[PT + 2 * S];
#pragma unroll
    for (int d = 0; d < S; ++d) x[d] = gl[d];
#pragma unroll
    for (int e = 0; e < PT; ++e) x[S + e] = v[e];
    x[S + PT - 1] = is_short ? gr[0] : v[PT - 1];
#pragma unroll
    for (int d = 0; d < S; ++d) {
      const Real full = gr[d], shrt = d + 1 < S ? gr[d + 1] : gr[d];
      x[S + PT + d] = is_short ? shrt : full;
    }
    // x_{i+o} - x_i serves point i and, negated (exactly), point i + o
    Real dn[S + 1][S + 1];   // dn[o][j] = x_{e-j+o} - x_{e-j}, j = 1..o: differences seen from below
#pragma unroll
    for (int o = 1; o <= S; ++o)
#pragma unroll
      for (int j = 1; j <= o; ++j) dn[o][j] = x[S - j + o] - x[S - j];
#pragma unroll
    for (int e = 0; e < PT; ++e) {
      const Real u0 = x[S + e];
      Real up[S + 1];
#pragma unroll
      for (int o = 1; o <= S; ++o) up[o] = x[S + e + o] - u0;
      if constexpr (EQ == AT_ADVDIFF) {
        Real a = Real(0);
#pragma unroll
        for (int o = 1; o <= S; ++o) a = add_pair(a, kad[S - o], -dn[o][o], kad[S + o], up[o]);
        put(e, u0, a);
      } else {
        Real l = Real(0), g = Real(0);
#pragma unroll
        for (int o = 1; o <= S; ++o) {
          l = add_pair(l, lap[S - o], -dn[o][o], lap[S + o], up[o]);
          g = add_pair(g, grd[S - o], -dn[o][o], grd[S + o], up[o]);
        }
        put(e, u0, burgers_rhs(u0, l, g));
      }
#pragma unroll
      for (int o = 1; o <= S; ++o) {
#pragma unroll
        for (int j = o; j > 1; --j) dn[o][j] = dn[o][j - 1];
        dn[o][1] = up[o];
      }
      if (kLong && !FG && (e & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
  };

  const int batch = line_batch(faces);
  int par = 0;
  int r0 = nslots > 0 ? mod_small(n0, nslots) : 0;
  // The delays are drawn two steps ahead of their use at least: batch j (steps
  // j batch ..) into half j & 1 during step j batch - 2, whose threads have all
  // read what that half held before the barrier that began it.
  int row = 0, half = 0;     // of the step after the current one
  // (A batch is two steps at least. The single-step form is kept in the text:
  // without it the compiler lays the step loop out otherwise, 256 points 0.50 ->
  // 0.515 us a step, the ensemble of 512 members 1.51 -> 1.53 ms.)
  for (int64_t nb = 0; nb < nsteps && nb < 2; nb += batch)
    draw(n0 + nb, static_cast<int>(nsteps - nb < batch ? nsteps - nb : batch), static_cast<int>(nb & 1));
  // steps until the next batch is drawn (batch j begins at step j batch), and
  // the half it goes to
  int until = batch == 1 ? 1 : batch - 1, next_half = batch == 1 ? 0 : 1;
  if (active) put_edges(u, s_e);
  __syncthreads();
  int k = active ? delays_at(0, 0) : 0;
  Real hl[S], hr[S];         // halos of the coming step (faces with a delay)
  Raw nl, nr;                // Heun: the next step's levels, read in its first stage
  int k_next = 0;
#pragma unroll
  for (int d = 0; d < S; ++d) hl[d] = hr[d] = Real(0);
  if (active) {
    Raw ql, qr_;
    halo_raw(0, ring, r0, k & 0xff, ql);
    halo_raw(1, ring, r0, k >> 8, qr_);
    halo_sum(k & 0xff, ql, hl);
    halo_sum(k >> 8, qr_, hr);
  }
  __syncthreads();           // the first row of delays is read before it is drawn over
  for (int64_t st = 0; st < nsteps; ++st) {
    const int64_t n = n0 + st;
    const int rn = r0 + 1 == nslots ? 0 : r0 + 1;
    if (++row == batch) {
      row = 0;
      half ^= 1;
    }
    const Real* e_in = s_e + par * eset;
    Real* e_out = s_e + (par ^ 1) * eset;
    if (active) {
      // the next step's halos: every level they take is published, so their
      // reads are off this step's chain (long chunks issue them late, when
      // registers are free)
      const int kn = st + 1 < nsteps ? delays_at(row, half) : 0;
      Raw ql, qr_;
      auto next_raw = [&]() __attribute__((always_inline)) {
        halo_raw(0, ring, rn, kn & 0xff, ql);
        halo_raw(1, ring, rn, kn >> 8, qr_);
      };
      Real fo[FG ? kAhead : 1][4];
      if constexpr (FG)
#pragma unroll
        for (int g = 0; g < kAhead; ++g) get4(g, fo[g]);
      if constexpr (kLate < 0) next_raw();
      Real gl[S], gr[S];
      ghosts(e_in, k, hl, hr, gl, gr);
      if constexpr (kRk2) {
        Real* e_star = s_e + 2 * eset + par * eset;
        // the predictor's halos (levels n - k - m < n of u*)
        Raw sl, sr;
        halo_raw(0, sring, r0, k & 0xff, sl);
        halo_raw(1, sring, r0, k >> 8, sr);
        stencil(u, gl, gr, [&](int e, Real u0, Real f) __attribute__((always_inline)) { us[e] = euler_update(u0, dt, f); });
        put_edges(us, e_star);
        publish(us, sring, r0);
        halo_sum(k & 0xff, sl, hl);
        halo_sum(k >> 8, sr, hr);
      } else if constexpr (KIND == AT_EULER) {
        stencil(u, gl, gr, [&](int e, Real u0, Real f) __attribute__((always_inline)) {
          if (e == kLate) next_raw();
          u[e] = euler_update(u0, dt, f);
        });
      } else if constexpr (KIND == AT_AB2) {
        // Euler at n = 0 (f^{-1} is taken as zero)
        const Real b1 = n > 0 ? Real(1.5) : Real(1), b2 = n > 0 ? Real(-0.5) : Real(0);
        if constexpr (FG) {
          // four groups of history in flight ahead of the stencil
          stencil(u, gl, gr, [&](int e, Real u0, Real f) __attribute__((always_inline)) {
            const int g = e >> 2;
            if (e == kLate) next_raw();
            u[e] = ab2_update(u0, dt, b1, f, b2, fo[g % kAhead][e & 3]);
            fo[g % kAhead][e & 3] = f;
            if ((e & 3) == 3) {
              put4(g, fo[g % kAhead]);
              if (g + kAhead < PT / 4) get4(g + kAhead, fo[g % kAhead]);
              __builtin_amdgcn_sched_barrier(0);
            }
          });
        } else {
          stencil(u, gl, gr, [&](int e, Real u0, Real f) __attribute__((always_inline)) {
            if (e == kLate) next_raw();
            u[e] = ab2_update(u0, dt, b1, f, b2, fa[e]);
            fa[e] = f;
          });
        }
      } else {
        const Ab3<Real> c(n);
        stencil(u, gl, gr, [&](int e, Real u0, Real f) __attribute__((always_inline)) {
          u[e] = ab3_update(u0, dt, c, f, fa[e], fb[e]);
          fb[e] = fa[e];
          fa[e] = f;
        });
      }
      if constexpr (!kRk2) {
        if constexpr (kLong) {
          // (in this order the long forms fit their registers)
          if constexpr (kLate == PT) next_raw();
          halo_sum(kn & 0xff, ql, hl);
          halo_sum(kn >> 8, qr_, hr);
          __builtin_amdgcn_sched_barrier(0);
          put_edges(u, e_out);
          publish(u, ring, rn);
        } else {
          put_edges(u, e_out);
          publish(u, ring, rn);
          halo_sum(kn & 0xff, ql, hl);
          halo_sum(kn >> 8, qr_, hr);
        }
        k = kn;
      } else {
        // second stage after the predictor's edges are complete: below
        nl = ql;
        nr = qr_;
        k_next = kn;
      }
    }
    if constexpr (kRk2) {
      __syncthreads();
      if (active) {
        Real gl[S], gr[S];
        ghosts(s_e + 2 * eset + par * eset, k, hl, hr, gl, gr);
        stencil(us, gl, gr, [&](int e, Real u0, Real f) __attribute__((always_inline)) { u[e] = heun_update(u[e], u0, dt, f); });
        put_edges(u, e_out);
        publish(u, ring, rn);
        halo_sum(k_next & 0xff, nl, hl);
        halo_sum(k_next >> 8, nr, hr);
        k = k_next;
      }
    }
    // draw the batch that starts two steps on
    if (--until == 0) {
      until = batch;
      const int64_t left = nsteps - st - 2;
      if (left > 0) draw(n + 2, static_cast<int>(left < batch ? left : batch), next_half);
      next_half ^= 1;
    }
    __syncthreads();
    par ^= 1;
    r0 = rn;
  }

  // the state back to device memory
  const int64_t n1 = n0 + nsteps;
  if (!sync && !GR)
    for (int i = tid; i < rtotal; i += nt) {
      B.ring[i] = s_ring[i];
      if (kRk2) B.sring[i] = s_sring[i];
    }
  // (the last point of a short chunk belongs to the next one)
  auto put_field = [&](Real* dst, const Real* v) __attribute__((always_inline)) {
    if (!active) return;
#pragma unroll
    for (int e = 0; e < PT - 1; ++e) dst[off + e] = v[e];
    if (!is_short) dst[off + PT - 1] = v[PT - 1];
  };
  if constexpr (kAb) {
    Real* f1p = KIND == AT_AB3 ? (((n1 - 1) & 1) ? B.f1 : B.f0) : B.f0;
    Real* f2p = KIND == AT_AB3 ? ((n1 & 1) ? B.f1 : B.f0) : nullptr;
    if constexpr (FG) {
      if (active)
#pragma unroll 4
        for (int g = 0; g < PT / 4; ++g) {
          Real v[4];
          get4(g, v);
#pragma unroll
          for (int j = 0; j < 4; ++j) f1p[off + 4 * g + j] = v[j];
        }
      __syncthreads();   // the transposed history is read before u_out takes u
    } else {
      put_field(f1p, fa);
    }
    if constexpr (KIND == AT_AB3)
      if (n1 > 1) put_field(f2p, fb);
  }
  put_field(B.u_out, u);
  if constexpr (kRk2) put_field(B.ustar, us);
  __syncthreads();   // LDS is free for the next line
}

}  // namespace atfd
