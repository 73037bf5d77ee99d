// Shared by the gathering stage kernels of the adjoint (adjoint2d.hpp for 1-D
// and 2-D, adjoint3d.hpp for 3-D; adjoint.hip states the method and the
// formula). One workgroup does everything a stage does for a PE, and every
// value is gathered:
//  - the forward halo values (for the Laplacian and the gradient of the stage
//    field) are the forward step's own combinations, read from the segment's
//    ring, whose slots keep every level of the segment;
//  - the transposed taps that leave a PE across a face with a delay go, once,
//    to the g ring: g_n[entry] = sum K mu over the consumer's points, in the
//    ring slot of step n at the neighbour's strip entry;
//  - the adjoint of level n of a strip entry is then the sum over the later
//    steps n' = n + j whose delay k' reaches level n (0 <= j - k' < T) of
//    c_{j-k'}(k') g_{n'}, and, where the neighbour's delay at n is 0, of the
//    neighbour's taps themselves. No ring entry is read and written back, or
//    cleared; the sums are in double.
#pragma once

#include <type_traits>

#include "adjoint.hpp"

namespace atfd {
namespace adjg {

constexpr int kDrain = 6;        // g values of an entry read ahead (more: a loop)
constexpr int kMaxDrain = 15;    // steps n + 1 .. n + 15 (at most L + T - 2 = 10 reach level n)

template <typename Real>
struct Two {
  Real v[2];
};

// Two consecutive values; EVEN: PE x edges are even, so both exist; else the
// second repeats the first past the PE's row.
template <bool EVEN, typename Real>
__device__ __forceinline__ Two<Real> ld2(const Real* p, bool has2) {
  Two<Real> r;
  if constexpr (EVEN) {
    __builtin_memcpy(&r, p, sizeof(r));
  } else {
    r.v[0] = p[0];
    r.v[1] = p[has2 ? 1 : 0];
  }
  return r;
}
template <bool EVEN, typename Real>
__device__ __forceinline__ void st2(Real* p, const Two<Real>& q, bool has2) {
  if constexpr (EVEN) {
    __builtin_memcpy(p, &q, sizeof(q));
  } else {
    p[0] = q.v[0];
    if (has2) p[1] = q.v[1];
  }
}

// Delay of face f of PE pid at step n (the synchronous scheme: 0).
__device__ __forceinline__ int delay_of(const StepParams& p, int pid, int f, int64_t n) {
  int k = 0;
  if (p.mode == AT_DELAY_RNG)
    k = raw_delay(p.key, n, static_cast<uint32_t>(pid * 2 * p.ndim + f), p.thr, p.L);
  else if (p.mode == AT_DELAY_HOST)
    k = p.host_delays[(n * p.npe + pid) * (2 * p.ndim) + f];
  else
    return 0;
  return clamp_startup(k, n, p.T);
}

// A kernel parameter into a register, opaque to the compiler: a choice between
// parameters is otherwise turned into a read at a chosen address, a memory
// latency that the address after it waits for.
__device__ __forceinline__ int64_t held(int64_t v) {
  asm("" : "+v"(v));
  return v;
}

// Strips in a ring (ring_index): element r of plane z of face f of PE e in slot
// s lies at strip0(f, e, slots, r) + s slot_step(f) + z strip_zs(f, slots).
__device__ __forceinline__ int64_t chunk_of(const StepParams& p, int f) {
  const int64_t a = held(p.face_chunk[0]), b = held(p.face_chunk[2]), c = held(p.face_chunk[4]);
  return f < 2 ? a : f < 4 ? b : c;
}
__device__ __forceinline__ int64_t foff_of(const StepParams& p, int f) {
  const int64_t o0 = held(p.face_off[0]), o1 = held(p.face_off[1]), o2 = held(p.face_off[2]),
                o3 = held(p.face_off[3]), o4 = held(p.face_off[4]), o5 = held(p.face_off[5]);
  return f == 0 ? o0 : f == 1 ? o1 : f == 2 ? o2 : f == 3 ? o3 : f == 4 ? o4 : o5;
}
__device__ __forceinline__ int64_t strip0(const StepParams& p, int f, int e, int slots, int64_t r) {
  const int64_t k = p.pe_major ? slots : 1;
  return k * foff_of(p, f) + e * k * chunk_of(p, f) + r;
}
__device__ __forceinline__ int64_t slot_step(const StepParams& p, int f) {
  const int64_t all = static_cast<int64_t>(p.npe) * held(p.pe_block), c = chunk_of(p, f);
  return p.pe_major ? c : all;
}
__device__ __forceinline__ int64_t strip_zs(const StepParams& p, int f, int slots) {
  return static_cast<int64_t>(p.npe) * chunk_of(p, f) * (p.pe_major ? slots : 1);
}

// What a stage needs of the PE's faces (LDS): neighbours and this PE's delays;
// the forward combination of the stage field across face f (weights, offsets
// of the slots in the neighbour's strip; a level of weight zero re-reads level
// n - k); the entries of the g ring that reach level n (weights, offsets of the
// slots in this PE's strip, zero past the count), and whether the neighbour's
// delay at n is 0; the taps by |o| (0 beyond S), [o > 0][|o|]: t1 = alpha c2
// (Burgers) or kad, t2 = c1 (Burgers).
template <int S, int TT, int NF>
struct Faces {
  int64_t hoff[NF][TT], goff[NF][kMaxDrain];
  double w[NF][TT], dw[NF][kMaxDrain];
  double t1[3][2][2 * S + 1], t2[3][2][2 * S + 1];
  // element 0 of plane 0 of: the neighbour's strip in the forward ring (slot 0),
  // this PE's strip in the g ring (slot 0), the neighbour's in step n's slot
  int64_t hbase[NF], gbase[NF], pbase[NF];
  int nbr[NF], k[NF], own[NF], cnt[NF];
};

// Fills fc; ends with a barrier. The draws of all faces and later steps run side
// by side, each on one lane and on registers only (weights are computed, not
// read from a table: a chain of reads at run-time addresses took longer than
// the rest of a 2-D stage's set-up); at least 192 threads.
template <int S, int TT, int NF, bool BURG>
__device__ __forceinline__ void face_setup(const AdjParams& q, int pe, Faces<S, TT, NF>& fc) {
  const StepParams& p = q.sp;
  const int tid = threadIdx.x;
  const int64_t n = q.n;
  const bool sync = p.mode == AT_SYNC;
  const int T = sync ? 1 : p.T;
  if (tid < 16 * NF + NF) {
    // lanes of the first kind: step n + j of the neighbour's face across f;
    // of the second: step n of face f itself
    const bool later = tid < 16 * NF;
    const int f = later ? tid >> 4 : tid - 16 * NF, j = later ? tid & 15 : 0;
    const int64_t nn = n + j;
    const int nb = neighbour(p, pe, f);
    const bool use = !later || (j <= (sync ? 0 : p.L + T - 2) && nn < q.nsteps);
    const int k = use ? delay_of(p, later ? nb : pe, later ? f ^ 1 : f, nn) : 0;
    double wk[kMaxT];
    level_weights(k, T, wk);
    if (later) {
      const int m = j - k;
      double w = 0.0;
#pragma unroll
      for (int i = 0; i < kMaxT; ++i) w = m == i && i < T && use ? wk[i] : w;
      // the 16 lanes of a face compact their entries; j = 0 is the neighbour's
      // own step (weight 1 where its delay is 0), the rest follow in order
      const uint64_t live = __ballot(j > 0 && w != 0.0);
      const uint32_t group = static_cast<uint32_t>(live >> ((tid & 63) & ~15)) & 0xffffu;
      const uint32_t below = group & ((1u << j) - 1u);
      const int cnt = __popc(group);
      if (j == 0) {
        fc.own[f] = w != 0.0;
        fc.cnt[f] = cnt;
      } else {
        const bool on = w != 0.0;
        int slot = q.gslot + j;
        while (slot >= q.anslots) slot -= q.anslots;   // (anslots = 1: the synchronous arm)
        const int at = on ? __popc(below) : cnt + (j - 1) - __popc(below);
        fc.dw[f][at] = w;
        fc.goff[f][at] = on ? slot * slot_step(p, f) : 0;
      }
    } else {
      fc.nbr[f] = nb;
      fc.k[f] = k;
      const int64_t step = slot_step(p, f ^ 1);
      fc.hbase[f] = strip0(p, f ^ 1, nb, q.fslots, 0);
      fc.gbase[f] = strip0(p, f, pe, q.anslots, 0);
      fc.pbase[f] = strip0(p, f ^ 1, nb, q.anslots, 0) + q.gslot * step;
#pragma unroll
      for (int m = 0; m < TT; ++m) {
        const double w = m < T ? wk[m] : 0.0;
        fc.w[f][m] = w;
        fc.hoff[f][m] = sync ? 0 : slot_back(q.fslot, k + (w != 0.0 ? m : 0), q.fslots) * step;
      }
    }
  }
  if (tid >= 128 && tid < 128 + 3 * 2 * (2 * S + 1)) {
    const int e = tid - 128;
    const int a = e / (2 * (2 * S + 1)), r = e - a * 2 * (2 * S + 1), up = r >= 2 * S + 1, o = up ? r - (2 * S + 1) : r;
    const bool in = o <= S;
    const int at = in ? (up ? S + o : S - o) : 0;
    fc.t1[a][up][o] = !in ? 0.0 : BURG ? p.alpha * p.c2[a][at] : p.kad[a][at];
    fc.t2[a][up][o] = !in || !BURG ? 0.0 : p.c1[a][at];
  }
  __syncthreads();
}

// The transposed taps of the points ia = 0 .. S - 1 counted from a face of axis
// a into the point at distance e across it (up: towards larger coordinates); mu
// and, for Burgers, pr = c mu at those points.
template <int S, int TT, int NF, bool BURG>
__device__ __forceinline__ double face_taps(const Faces<S, TT, NF>& fc, int a, int up, int e, const double (&mu)[S],
                                   const double (&pr)[S]) {
  double g = 0.0;
#pragma unroll
  for (int ia = 0; ia < S; ++ia) {
    g += fc.t1[a][up][1 + e + ia] * mu[ia];
    if (BURG) g -= fc.t2[a][up][1 + e + ia] * pr[ia];
  }
  return g;
}

}  // namespace adjg
}  // namespace atfd
