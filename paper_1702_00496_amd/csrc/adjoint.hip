// Discrete adjoint of the AT time step (advection-diffusion or viscous
// Burgers; Euler, AB2 or Heun RK2).
//
// One stage of the forward step computes, at every point i from a stage field
// c (u for Euler/AB2 and the first RK2 stage, the predictor u* for the second),
//   F_i = alpha sum_{a,o} c2_o (v_{a,o} - c_i) - [c . grad] ,
// where v_{a,o} = c_{i+o} for a tap inside the PE of i (Sec. 2 eq.
// general_deriv) and, for a tap across face f, the AT combination
// sum_m c_m(k) c^{n-k-m}_{i+o} of that field's history with the face's delay k
// (Sec. 3.4 Example 3 eq. cd4-at); the advection term is sum c_a c1_o (v - c_i)
// (advection-diffusion) or c_i sum c1_o (v - c_i) (Burgers; Sec. 5 eq.
// general). Linearised, dF_i = sum K_{i,a,o} dv_{a,o} + D_i dc_i with
//   K_{i,a,o} = alpha c2_o - c_a c1_o  or  alpha c2_o - c_i c1_o,
//   D_i = -sum K_{i,a,o}  (- G_i = -sum c1_o (v - c_i) for Burgers).
// Given mu = dJ/dF (one field), the stage adjoint is
//   out_j = (base terms) + D_j mu_j + sum_{o: j-o in the PE of j} K_{j-o,a,o} mu_{j-o} + A^n_j,
// where A^l gathers, at the edge strips that neighbours read, K_{i,a,o} c_m(k)
// mu_i of every later step with n - k - m = l: an adjoint ring of the forward
// ring's shape, filled in gather form (one thread per strip value: the strip
// kernel) and drained when the sweep reaches level l. 1-D, 2-D and most 3-D
// problems take the stage kernels of adjoint2d.hpp and adjoint3d.hpp instead,
// which keep the sums over mu themselves and combine them when level l is
// reached; the kernels here, whose grid is the points and strip values, serve
// 3-D problems of few, deep or very small PEs (adj3d_pays) and the shapes the
// others cannot hold (3-D cross-sections of more than 2048 points, planes too
// large for LDS). They take both field layouts. The alpha-gradient adds
// <mu, dF/dalpha> = <mu, AT Laplacian of c>.
//
// Euler/AB2 (Sec. 4.1 eqs. time_disc, time_ab2): one stage per step, mu =
// dt (beta0 lambda^{n+1} + beta1 lambda^{n+2}), out = lambda^n with base
// lambda^{n+1}. Heun: stage 2 with mu = dt/2 lambda^{n+1} gives sigma = dJ/du*
// (base lambda^{n+1}/2, predictor ring), then stage 1 with mu = dt sigma gives
// lambda^n (base lambda^{n+1}/2 + sigma, solution ring).

#include "adjoint.hpp"

#include <algorithm>
#include <type_traits>

namespace atfd {
namespace {

constexpr int kAdjThreads = 256;

struct Pt {
  int pe;           // PE id
  int l[3];         // coordinates inside the PE
};

// Field index of the point at PE coordinates (x, y, z) of PE pe, in either
// field layout.
__device__ inline int64_t cell(const StepParams& p, int pe, int x, int y, int z) {
  if (p.pe_major) return ((static_cast<int64_t>(pe) * p.bz + z) * p.by + y) * p.bx + x;
  const int r = pe / p.px, qz = r / p.py, qx = pe - r * p.px, qy = r - qz * p.py;
  return ((static_cast<int64_t>(qz) * p.bz + z) * p.ny + static_cast<int64_t>(qy) * p.by + y) * p.nx +
         static_cast<int64_t>(qx) * p.bx + x;
}

// The point at field index g (fields below 2^31 points: the host checks).
__device__ inline Pt point_of(const StepParams& p, int64_t g64) {
  Pt r;
  const uint32_t g = static_cast<uint32_t>(g64);
  const uint32_t nx = static_cast<uint32_t>(p.pe_major ? p.bx : p.nx), ny = static_cast<uint32_t>(p.pe_major ? p.by : p.ny);
  const uint32_t row = g / nx;
  const int x = static_cast<int>(g - row * nx), z = static_cast<int>(row / ny);
  const int y = static_cast<int>(row - static_cast<uint32_t>(z) * ny);
  const int qz = z / p.bz;
  r.l[2] = z - qz * p.bz;
  if (p.pe_major) {   // z counts planes through all PEs
    r.l[0] = x;
    r.l[1] = y;
    r.pe = qz;
    return r;
  }
  const int qx = x / p.bx, qy = y / p.by;
  r.l[0] = x - qx * p.bx;
  r.l[1] = y - qy * p.by;
  r.pe = qx + p.px * (qy + p.py * qz);
  return r;
}

__device__ inline int edge_of(const StepParams& p, int a) { return a == 0 ? p.bx : a == 1 ? p.by : p.bz; }

// Component a of a 3-vector, and a write of it, by selects: a run-time index
// into a local array would put the array in scratch memory.
__device__ inline int sel3(int a, int v0, int v1, int v2) { return a == 0 ? v0 : a == 1 ? v1 : v2; }
__device__ inline void set3(int* l, int a, int v) {
  l[0] = a == 0 ? v : l[0];
  l[1] = a == 1 ? v : l[1];
  l[2] = a == 2 ? v : l[2];
}

// Element of the strip of face F = 2a + side of a PE for the point with PE
// coordinates l (which must lie in that strip): x faces [z][y][d], y faces
// [z][d][x], z faces [d][y][x], with depth d counted from the PE's low side.
__device__ inline int64_t strip_elem(const StepParams& p, int F, const int* l, int S) {
  const int a = F >> 1;
  const int b = edge_of(p, a);
  const int la = sel3(a, l[0], l[1], l[2]);
  const int d = (F & 1) ? la - (b - S) : la;
  if (a == 0) return (static_cast<int64_t>(l[2]) * p.by + l[1]) * S + d;
  if (a == 1) return (static_cast<int64_t>(l[2]) * S + d) * p.bx + l[0];
  return (static_cast<int64_t>(d) * p.by + l[1]) * p.bx + l[0];
}

// Index, in a ring of ns slots, of the strip value of face F at PE coordinates l
// (in that strip): x faces plane z, [y][d]; y faces plane z, [d][x]; z faces
// plane d, [y][x].
__device__ inline int64_t ring_at_pt(const StepParams& p, int ns, int slot, int pe, int F, const int* l, int S) {
  const int a = F >> 1;
  const int b = edge_of(p, a);
  const int la = sel3(a, l[0], l[1], l[2]);
  const int d = (F & 1) ? la - (b - S) : la;
  if (a == 0) return ring_index(p, ns, slot, pe, F, l[2], static_cast<int64_t>(l[1]) * S + d);
  if (a == 1) return ring_index(p, ns, slot, pe, F, l[2], static_cast<int64_t>(d) * p.bx + l[0]);
  return ring_index(p, ns, slot, pe, F, d, static_cast<int64_t>(l[1]) * p.bx + l[0]);
}

// Strip value t of the per-PE numbering used by the strip kernel
// and the halo buffer: PE pe, face F (its strip starts at pfo[F] inside the
// PE's pe_block values), depth d from the strip's low side and the other PE
// coordinates in l (l[F >> 1] = 0). 32-bit: the host keeps npe * pe_block
// below 2^31.
struct StripPt {
  int pe, F, d;
  int l[3];
};

template <int S>
__device__ inline StripPt strip_point(const AdjParams& q, int t) {
  const StepParams& p = q.sp;
  const int blk = static_cast<int>(p.pe_block);
  StripPt s;
  s.pe = t / blk;
  const int r = t - s.pe * blk;
  int F = 0, off = 0;
#pragma unroll
  for (int f = 1; f < 6; ++f) {
    const bool past = f < 2 * p.ndim && r >= static_cast<int>(q.pfo[f]);
    F += past ? 1 : 0;
    off = past ? static_cast<int>(q.pfo[f]) : off;
  }
  s.F = F;
  const int e = r - off;
  const int a = F >> 1;
  s.l[0] = s.l[1] = s.l[2] = 0;
  if (a == 0) {
    s.d = e % S;
    s.l[1] = (e / S) % p.by;
    s.l[2] = e / (p.by * S);
  } else if (a == 1) {
    s.l[0] = e % p.bx;
    s.d = (e / p.bx) % S;
    s.l[2] = e / (p.bx * S);
  } else {
    s.l[0] = e % p.bx;
    s.l[1] = (e / p.bx) % p.by;
    s.d = e / (p.bx * p.by);
  }
  return s;
}

__device__ inline int nbr_pe(const StepParams& p, int pid, int f) {
  int q[3] = {pid % p.px, (pid / p.px) % p.py, pid / (p.px * p.py)};
  const int a = f >> 1;
  const int ext = sel3(a, p.px, p.py, p.pz);
  set3(q, a, (sel3(a, q[0], q[1], q[2]) + ((f & 1) ? 1 : ext - 1)) % ext);
  return q[0] + p.px * (q[1] + p.py * q[2]);
}

// Delay of face f of PE pid at step n; the synchronous scheme is k = 0 with
// a single level.
__device__ inline int adj_delay(const StepParams& p, int pid, int f, int64_t n) {
  int k = 0;
  if (p.mode == AT_DELAY_RNG)
    k = raw_delay(p.key, n, static_cast<uint32_t>(pid * 2 * p.ndim + f), p.thr, p.L);
  else if (p.mode == AT_DELAY_HOST)
    k = p.host_delays[(n * p.npe + pid) * (2 * p.ndim) + f];
  else
    return 0;
  return clamp_startup(k, n, p.T);
}

__device__ inline int adj_levels(const StepParams& p) { return p.mode == AT_SYNC ? 1 : p.T; }

// mu = dJ/dF of this stage at point g: m0 y0 + m1 y1, formed where it is
// used. Without a second field (m1 = 0) y1 falls back to y0, so both loads
// are unconditional and the m1 term is an exact zero for finite y0.
template <typename Real>
__device__ inline double mu_at(const AdjParams& q, int64_t g) {
  const Real* y0 = static_cast<const Real*>(q.y0);
  const Real* y1 = static_cast<const Real*>(q.m1 != 0.0 ? q.y1 : q.y0);
  return q.m0 * static_cast<double>(y0[g]) + q.m1 * static_cast<double>(y1[g]);
}

template <typename Real>
__device__ inline double centre_at(const AdjParams& q, int64_t g) {
  return static_cast<double>(static_cast<const Real*>(q.levels)[(q.n - q.seg_start) * q.npts + g]);
}

// Tap K_{i,a,o} at a consumer point with stage value ci.
__device__ inline double tap_k(const AdjParams& q, int a, int o, double ci) {
  const StepParams& p = q.sp;
  if (q.burgers) return p.alpha * p.c2[a][o + p.s] - ci * p.c1[a][o + p.s];
  return p.kad[a][o + p.s];
}

// Scatter of step n (gather form): every strip value e of face F of PE q
// collects the transposed taps of the consumer PE across F, weighted by the
// consumer's level weights, into the adjoint ring slots of levels n-k-m.
template <typename Real, int S>
__device__ inline void scatter_elem(const AdjParams& q, const StripPt& sp, const double (*wt)[kMaxT]) {
  const StepParams& p = q.sp;
  double* aring = static_cast<double*>(q.aring);
  const int pe = sp.pe, F = sp.F, d = sp.d, a = F >> 1;
  const int* l = sp.l;
  const int b = edge_of(p, a);
  // the consumer across F reads this strip through its opposite face
  const int cons = nbr_pe(p, pe, F);
  const int cf = F ^ 1;
  // coordinate of the strip value in the consumer's frame
  const int jp = (F & 1) ? d - S : b + d;
  // taps from consumer points outside the consumer PE are dropped by a
  // select after unconditional loads from a clamped (in-PE) point, so that
  // every load of the element is in flight together
  double g = 0.0;
#pragma unroll
  for (int o = -S; o <= S; ++o) {
    if (o == 0) continue;
    const int ia = jp - o;
    const bool valid = ia >= 0 && ia < b;
    int c[3] = {l[0], l[1], l[2]};
    set3(c, a, min(max(ia, 0), b - 1));
    const int64_t gi = cell(p, cons, c[0], c[1], c[2]);
    const double ci = q.burgers ? centre_at<Real>(q, gi) : 0.0;   // Burgers taps only
    const double t = tap_k(q, a, o, ci) * mu_at<Real>(q, gi);
    g += valid ? t : 0.0;
  }
  const int k = adj_delay(p, cons, cf, q.n);
  const double* w = wt[k];
  const int T = adj_levels(p);
  int lsF[3] = {l[0], l[1], l[2]};   // the strip value's PE coordinates
  set3(lsF, a, (F & 1) ? b - S + d : d);
  double* dst[kMaxT];
  double old[kMaxT];
#pragma unroll
  for (int m = 0; m < kMaxT; ++m) {
    if (m >= T) break;
    // level n - k - m (before t = 0 only where w[m] = 0: any slot is read)
    const int slot = slot_back(q.gslot, k + m, q.anslots);
    dst[m] = aring + ring_at_pt(p, q.anslots, slot, pe, F, lsF, S);
    old[m] = *dst[m];
  }
#pragma unroll
  for (int m = 0; m < kMaxT; ++m) {
    if (m >= T) break;
    if (w[m] != 0.0) *dst[m] = old[m] + w[m] * g;
  }
}

// The forward halo values of step n, for the alpha-derivative: for every
// consumer PE, face f and element e of the producer strip it reads, the AT
// combination of the segment's ring (the synchronous scheme: level n).
// hbuf[pe * pe_block + (per-PE offset of face f) + e].
template <typename Real, int S>
__device__ inline Real halo_value(const AdjParams& q, const StripPt& sp, const double (*wt)[kMaxT]) {
  const StepParams& p = q.sp;
  const int T = adj_levels(p);
  const int pe = sp.pe, f = sp.F, d = sp.d, a = f >> 1, pf = f ^ 1;
  int ls[3] = {sp.l[0], sp.l[1], sp.l[2]};
  const int b = edge_of(p, a);
  set3(ls, a, (pf & 1) ? b - S + d : d);
  const int src = nbr_pe(p, pe, f);
  const int k = adj_delay(p, pe, f, q.n);
  const double* w = wt[k];
  if (p.mode == AT_SYNC)   // level n, always stored
    return static_cast<const Real*>(q.levels)[(q.n - q.seg_start) * q.npts + cell(p, src, ls[0], ls[1], ls[2])];
  // all kMaxT levels are loaded unconditionally (a level m >= T repeats
  // level T - 1 and is dropped below, like a level of weight zero), so the
  // loads overlap
  const Real* R = static_cast<const Real*>(q.fring);
  double lv[kMaxT];
#pragma unroll
  for (int m = 0; m < kMaxT; ++m)
    lv[m] = static_cast<double>(R[ring_at_pt(p, q.fslots, slot_back(q.fslot, k + min(m, T - 1), q.fslots), src, pf, ls, S)]);
  double v = 0.0;
#pragma unroll
  for (int m = 0; m < kMaxT; ++m)
    if (m < T && w[m] != 0.0) v += w[m] * lv[m];
  return static_cast<Real>(v);
}

template <typename Real, int S>
__device__ inline void halo_elem(const AdjParams& q, int t, const StripPt& sp, const double (*wt)[kMaxT]) {
  static_cast<Real*>(q.hbuf)[t] = halo_value<Real, S>(q, sp, wt);
}

// One thread per strip value t: its forward halo value (consumer view) and its
// adjoint-ring scatter (producer view) share the decode of t.
template <typename Real, int S>
__global__ __launch_bounds__(kAdjThreads) void adj_strip_kernel(AdjParams q) {
  // the level weights c_m(k) of every delay k < L (the delays are clamped
  // below L), once per workgroup
  __shared__ double s_wt[kMaxL][kMaxT];
  if (threadIdx.x < kMaxL * kMaxT) s_wt[threadIdx.x / kMaxT][threadIdx.x % kMaxT] = q.wt[threadIdx.x / kMaxT][threadIdx.x % kMaxT];
  __syncthreads();
  const int total = q.sp.npe * static_cast<int>(q.sp.pe_block);
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < total; t += gridDim.x * blockDim.x) {
    const StripPt sp = strip_point<S>(q, t);
    halo_elem<Real, S>(q, t, sp, s_wt);
    scatter_elem<Real, S>(q, sp, s_wt);
  }
}

// The stage adjoint out = b0 x0 + b1 x1 + D mu + transposed taps + the adjoint
// ring slot of level n (drained and cleared here), plus this stage's part of
// dJ/dalpha. Branch-free per point: every lane issues the same loads, a tap
// that leaves the PE selects the address of its halo value (or of a value it
// then multiplies by zero), so PE-edge points cost what interior points cost.
template <typename Real, int DIM, int S>
__global__ __launch_bounds__(kAdjThreads) void adj_lambda_kernel(AdjParams q) {
  const StepParams& p = q.sp;
  Real* __restrict__ out = static_cast<Real*>(q.out);
  const Real* __restrict__ x0 = static_cast<const Real*>(q.x0);
  // with b1 = 0, x1 falls back to x0 (an exact zero term for finite x0)
  const Real* __restrict__ x1 = static_cast<const Real*>(q.b1 != 0.0 ? q.x1 : q.x0);
  const Real* __restrict__ C = static_cast<const Real*>(q.levels) + (q.n - q.seg_start) * q.npts;
  const Real* __restrict__ hb = static_cast<const Real*>(q.hbuf);
  double* __restrict__ aring = static_cast<double*>(q.aring);
  const int slot_n = q.gslot;
  // steps along the axes inside a PE
  const int64_t st[3] = {1, p.pe_major ? p.bx : p.nx,
                         p.pe_major ? static_cast<int64_t>(p.bx) * p.by : static_cast<int64_t>(p.nx) * p.ny};
  double da = 0.0;
  for (int64_t g = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; g < q.npts;
       g += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const Pt j = point_of(p, g);
    const double mu = mu_at<Real>(q, g);
    const double cj = static_cast<double>(C[g]);
    const double v1 = static_cast<double>(x1[g]);
    double acc = q.b0 * static_cast<double>(x0[g]) + q.b1 * v1;
    double lap = 0.0, grad = 0.0, sumk = 0.0;
    const Real* hpe = hb + static_cast<int64_t>(j.pe) * p.pe_block;
    // adjoint-ring entries of the strips j belongs to: every load of the
    // point is issued before the entries are cleared at the end
    double* rsrc[2 * DIM];
    bool rin[2 * DIM];
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      const int b = edge_of(p, a);
#pragma unroll
      for (int o = -S; o <= S; ++o) {
        if (o == 0) continue;
        sumk += tap_k(q, a, o, cj);
        // transposed interior tap: from i = j - o when i lies in the PE
        const int ia = j.l[a] - o;
        const bool tin = ia >= 0 && ia < b;
        const int64_t gi = tin ? g - o * st[a] : g;
        const double mi = mu_at<Real>(q, gi);
        // the stage value at i enters the Burgers taps only (uniform branch)
        const double ci = q.burgers ? static_cast<double>(C[gi]) : 0.0;
        acc += tin ? tap_k(q, a, o, ci) * mi : 0.0;
        // forward stencil of the stage field at j: inside the PE from the
        // field, across a face from the stage's combined halo values
        const int ta = j.l[a] + o;
        const bool fin = ta >= 0 && ta < b;
        const int side = ta < 0 ? 0 : 1;
        int ls[3] = {j.l[0], j.l[1], j.l[2]};
        ls[a] = fin ? (side ? b - S : 0) : (side ? ta - b : ta + b);
        const int f = 2 * a + side;
        const int64_t pfo = side ? q.pfo[2 * a + 1] : q.pfo[2 * a];   // uniform values, no indexed load
        const Real* pv = fin ? C + (g + o * st[a]) : hpe + pfo + strip_elem(p, f ^ 1, ls, S);
        const double v = static_cast<double>(*pv) - cj;
        lap += p.c2[a][o + S] * v;
        grad += p.c1[a][o + S] * v;
      }
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        const bool in = side ? j.l[a] >= b - S : j.l[a] < S;
        int ls[3] = {j.l[0], j.l[1], j.l[2]};
        if (!in) ls[a] = side ? b - S : 0;
        double* src = aring + ring_at_pt(p, q.anslots, slot_n, j.pe, 2 * a + side, ls, S);
        const double r = *src;
        acc += in ? r : 0.0;
        rsrc[2 * a + side] = src;
        rin[2 * a + side] = in;
      }
    }
#pragma unroll
    for (int f = 0; f < 2 * DIM; ++f)
      if (rin[f]) *rsrc[f] = 0.0;
    // D_j mu_j with D_j = -sum K (- G_j for Burgers)
    acc += (-sumk - (q.burgers ? grad : 0.0)) * mu;
    out[g] = static_cast<Real>(acc);
    da += mu * lap;
  }
  // fixed-order block reduction of the alpha-gradient part
  for (int off = 32; off > 0; off >>= 1) da += __shfl_down(da, off, 64);
  __shared__ double part[kAdjThreads / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x / 64] = da;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kAdjThreads / 64; ++w) s += part[w];
    q.partial[blockIdx.x] += s;
  }
}

template <typename Real>
hipError_t launch_strip(const AdjParams& q, int blocks, hipStream_t st) {
  switch (q.sp.s) {
    case 1: hipLaunchKernelGGL((adj_strip_kernel<Real, 1>), dim3(blocks), dim3(kAdjThreads), 0, st, q); break;
    case 2: hipLaunchKernelGGL((adj_strip_kernel<Real, 2>), dim3(blocks), dim3(kAdjThreads), 0, st, q); break;
    case 3: hipLaunchKernelGGL((adj_strip_kernel<Real, 3>), dim3(blocks), dim3(kAdjThreads), 0, st, q); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// (2-D and 3-D: a 1-D PE's line always fits the 1-D kernel's LDS)
template <typename Real>
hipError_t launch_lambda(const AdjParams& q, int blocks, hipStream_t st) {
  const int key = q.sp.ndim * 10 + q.sp.s;
  switch (key) {
#define ATFD_ADJ_CASE(D, S)                                                                         \
  case D * 10 + S:                                                                                   \
    hipLaunchKernelGGL((adj_lambda_kernel<Real, D, S>), dim3(blocks), dim3(kAdjThreads), 0, st, q); \
    break;
    ATFD_ADJ_CASE(2, 1) ATFD_ADJ_CASE(2, 2) ATFD_ADJ_CASE(2, 3)
    ATFD_ADJ_CASE(3, 1) ATFD_ADJ_CASE(3, 2) ATFD_ADJ_CASE(3, 3)
#undef ATFD_ADJ_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// One wave: lane l adds partials l, l + 64, ... in order, then a fixed
// butterfly combines the lanes.
__global__ __launch_bounds__(64) void adj_sum_kernel(const double* partial, int count, double* out) {
  double s = 0.0;
  for (int i = threadIdx.x; i < count; i += 64) s += partial[i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
  if (threadIdx.x == 0) out[0] = s;
}

}  // namespace

int adj_blocks(int64_t npts) {
  const int64_t b = (npts + kAdjThreads - 1) / kAdjThreads;
  return static_cast<int>(b < kAdjBlocks ? b : kAdjBlocks);
}

hipError_t launch_adj_step(const AdjParams& q, bool f64, hipStream_t st) {
  if (adj3d_applies(q.sp, f64)) return f64 ? launch_adj3d_f64(q, st) : launch_adj3d_f32(q, st);
  if (adj2d_applies(q.sp, f64)) {
    if (q.sp.ndim == 1) return f64 ? launch_adj1d_f64(q, st) : launch_adj1d_f32(q, st);
    return f64 ? launch_adj2d_f64(q, st) : launch_adj2d_f32(q, st);
  }
  const int64_t strips = static_cast<int64_t>(q.sp.npe) * q.sp.pe_block;
  const int64_t sb = (strips + kAdjThreads - 1) / kAdjThreads;
  const int sblocks = static_cast<int>(sb < kAdjBlocks ? (sb > 0 ? sb : 1) : kAdjBlocks);
  const hipError_t e = f64 ? launch_strip<double>(q, sblocks, st) : launch_strip<float>(q, sblocks, st);
  if (e != hipSuccess) return e;
  return f64 ? launch_lambda<double>(q, adj_blocks(q.npts), st) : launch_lambda<float>(q, adj_blocks(q.npts), st);
}

// Levels lo .. of one ring into another of a different slot count (grid y:
// level); a plain copy of slots, or of chunks where the slots are innermost.
template <typename Word>
__global__ __launch_bounds__(256) void ring_levels_kernel(StepParams p, const Word* __restrict__ src, int ns,
                                                          Word* __restrict__ dst, int nd, int64_t lo, uint32_t words,
                                                          int wsize) {   // wsize: values per word
  const int64_t l = lo + blockIdx.y;
  const int ss = static_cast<int>(l % ns), sd = static_cast<int>(l % nd);
  for (uint32_t w = blockIdx.x * blockDim.x + threadIdx.x; w < words; w += gridDim.x * blockDim.x) {
    if (!p.pe_major) {
      dst[static_cast<size_t>(sd) * words + w] = src[static_cast<size_t>(ss) * words + w];
      continue;
    }
    // [face][plane][pe][slot][chunk]: the chunk the word lies in
    int f = 0;
#pragma unroll
    for (int i = 1; i < 6; ++i) f += w >= static_cast<uint32_t>(p.face_off[i] / wsize) ? 1 : 0;
    const uint32_t fo = static_cast<uint32_t>((f == 0 ? p.face_off[0] : f == 1 ? p.face_off[1] : f == 2 ? p.face_off[2]
                        : f == 3 ? p.face_off[3] : f == 4 ? p.face_off[4] : p.face_off[5]) / wsize);
    const uint32_t chunk = static_cast<uint32_t>((f < 4 ? p.face_chunk[0] : p.face_chunk[4]) / wsize);
    const uint32_t blk = (w - fo) / chunk, r = (w - fo) - blk * chunk;
    const size_t so = static_cast<size_t>(ns) * fo + (static_cast<size_t>(blk) * ns + ss) * chunk + r;
    const size_t de = static_cast<size_t>(nd) * fo + (static_cast<size_t>(blk) * nd + sd) * chunk + r;
    dst[de] = src[so];
  }
}

hipError_t launch_ring_levels(const StepParams& p, bool f64, const void* src, int ns, void* dst, int nd, int64_t lo,
                              int64_t count, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  if (ns < 1 || nd < 1 || count > 65535) return hipErrorInvalidValue;
  const int w = f64 ? 8 : 4;
  const int64_t elems = static_cast<int64_t>(p.npe) * p.pe_block, bytes = elems * w;
  // 16-byte words where a slot (PE-major: every chunk) is a whole number of them
  const bool vec = p.pe_major ? (p.face_chunk[0] * w) % 16 == 0 && (p.face_chunk[4] * w) % 16 == 0 : bytes % 16 == 0;
  const int wb = vec ? 16 : w;
  const int64_t words = bytes / wb;
  if (words >= (int64_t(1) << 32)) return hipErrorInvalidValue;
  const unsigned blocks = static_cast<unsigned>(std::min<int64_t>((words + 255) / 256, 1024));
  const dim3 grid(blocks, static_cast<unsigned>(count));
  if (vec)
    hipLaunchKernelGGL((ring_levels_kernel<uint4>), grid, dim3(256), 0, st, p, static_cast<const uint4*>(src), ns,
                       static_cast<uint4*>(dst), nd, lo, static_cast<uint32_t>(words), 16 / w);
  else if (f64)
    hipLaunchKernelGGL((ring_levels_kernel<uint64_t>), grid, dim3(256), 0, st, p, static_cast<const uint64_t*>(src), ns,
                       static_cast<uint64_t*>(dst), nd, lo, static_cast<uint32_t>(words), 1);
  else
    hipLaunchKernelGGL((ring_levels_kernel<uint32_t>), grid, dim3(256), 0, st, p, static_cast<const uint32_t*>(src), ns,
                       static_cast<uint32_t*>(dst), nd, lo, static_cast<uint32_t>(words), 1);
  return hipGetLastError();
}

int adj_partials(const StepParams& p) { return p.npe > kAdjBlocks ? p.npe : kAdjBlocks; }

hipError_t launch_adj_sum(const double* partial, int count, double* out, hipStream_t st) {
  hipLaunchKernelGGL(adj_sum_kernel, dim3(1), dim3(64), 0, st, partial, count, out);
  return hipGetLastError();
}

}  // namespace atfd
