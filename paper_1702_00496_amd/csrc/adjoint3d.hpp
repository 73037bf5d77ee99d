// Stage of the reversed step for 3-D problems whose PEs fill the chip
// (adj3d_pays): one workgroup per PE, two x points per thread, sweeping the
// PE's z-planes (adjoint_gather.hpp: how the strips are done).
//
// What bounds it: FP64 issue and latency at two waves per SIMD. A neighbour pair
// takes up to nine FP64 operations and four conversions (Laplacian, gradient
// and the transposed sums, even and odd taps together). 256^3 in 8^3 PEs,
// sixth-order Burgers, FP32: 217 us a stage alone on the chip, the vector
// units busy 45 % of it (two rounds of 8 waves a CU, at 185 registers); 185 MiB
// are read and 80 MiB written, 53 us at the rate of a large copy. The separate
// strip kernel (read-modify-write of T ring slots from gathers strided by the
// row) and stage kernel (taps and products per tap through LDS) took 453 + 570
// us. 192^3 in 6^3 PEs, fourth-order AB2, 16 steps with the forward runs: 6.2 ->
// 2.4 ms. Two workgroups a CU at 128 registers spill: twice as slow (the forms
// of 1024 threads, which have no more, run at a third to a half of the rate of
// the others).

#pragma once

#include "adjoint_gather.hpp"

namespace atfd {
namespace adj3d {

using namespace adjg;

// MAXT: threads; TT: levels read of a combination (S + 1, the schemes' own
// count, or kMaxT for the others; weights past T are zero); BURG: Burgers (taps depend on the stage field); M1: mu has a
// second term (AB2).
template <typename Real, int S, int TT, bool BURG, bool M1, bool EVEN, int MAXT>
__global__ __launch_bounds__(MAXT) void adj3d_kernel(AdjParams q) {
  const StepParams& p = q.sp;
  using Y = typename std::conditional<M1, double, Real>::type;   // mu (M1), or y0 with m0 applied at the end
  using R2 = Two<Real>;
  constexpr int kCo = 4;                   // LDS column of x = 0
  constexpr int NT = 2 * S + 1;
  extern __shared__ __align__(16) unsigned char smem[];
  const int bx = p.bx, by = p.by, bz = p.bz;
  const int W = (bx + kCo + S + 2) & ~1, H = by + 2 * S;   // a quad of columns fits past the row
  const int plane = W * H;
  const int nxh = 2 * S * by, nh = nxh + 2 * S * bx;
  double* sA = reinterpret_cast<double*>(smem);              // [2][nh] drained entries
  Y* sY = reinterpret_cast<Y*>(sA + 2 * nh);                 // [2][plane]
  Real* sC = reinterpret_cast<Real*>(sY + 2 * plane);        // [2][plane]
  Real* sZ = sC + 2 * plane;                                 // [S][by][bx] planes bz .. bz + S - 1 of c
  __shared__ Faces<S, TT, 6> fc;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int pe = pe_of_workgroup(blockIdx.x, gridDim.x);
  const int64_t n = q.n;
  const bool sync = p.mode == AT_SYNC;
  const double m0 = q.m0, m1 = q.m1;

  // zero frames of mu
  for (int i = tid; i < 2 * plane; i += nt) sY[i] = Y(0);
  face_setup<S, TT, 6, BURG>(q, pe, fc);

  // ---- fields: plane z of PE e starts at e's base + z zs, rows pitch apart
  const int64_t pitch = p.pe_major ? bx : p.nx;
  const int64_t zs = p.pe_major ? static_cast<int64_t>(bx) * by : static_cast<int64_t>(p.nx) * p.ny;
  auto pe_base = [&](int e) __attribute__((always_inline)) -> int64_t {
    if (p.pe_major) return static_cast<int64_t>(e) * bx * by * bz;
    const PePos at = pe_pos(p, e);
    return (static_cast<int64_t>(at.z) * bz * p.ny + static_cast<int64_t>(at.y) * by) * p.nx + static_cast<int64_t>(at.x) * bx;
  };
  const Real* __restrict__ C = static_cast<const Real*>(q.levels) + (n - q.seg_start) * q.npts;
  const Real* __restrict__ Y0 = static_cast<const Real*>(q.y0);
  const Real* __restrict__ Y1 = static_cast<const Real*>(M1 ? q.y1 : q.y0);
  const Real* __restrict__ X0 = static_cast<const Real*>(q.x0);
  const bool b1 = q.b1 != 0.0;
  const Real* __restrict__ X1 = static_cast<const Real*>(b1 ? q.x1 : q.x0);
  Real* __restrict__ out = static_cast<Real*>(q.out);
  const Real* __restrict__ F = static_cast<const Real*>(q.fring);
  Real* G = static_cast<Real*>(q.aring);

  // ---- this thread's two points of a plane
  const int vx = (bx + 1) / 2;
  const bool active = tid < vx * by;
  const int y = active ? div_small(tid, vx) : 0, x = active ? 2 * (tid - y * vx) : 0;
  const bool has2 = EVEN || x + 1 < bx;
  const int64_t base = pe_base(pe);        // uniform
  const uint32_t col = static_cast<uint32_t>(y * pitch + x);
  const int at = (y + S) * W + kCo + x;

  // ---- this thread's item of the x / y frame: side and depth d of a face's
  // strip, line r. Beyond the face: the neighbour's strip pf, entry r (halo
  // value in, outgoing taps out); inside it: this PE's own strip f, entry r.
  const bool item = tid < nh;
  int f = 0, r = 0, d = 0, h_at = 0, in_at = 0, in_step = 0;
  if (item) {
    if (tid < nxh) {
      const int side = tid >= S * by ? 1 : 0;
      r = side ? tid - S * by : tid;
      const int yy = r / S;
      d = r - yy * S;
      f = side;
      h_at = (yy + S) * W + kCo + (side ? bx + d : d - S);
      in_at = (yy + S) * W + kCo + (side ? bx - 1 : 0);     // the point nearest the face
      in_step = side ? -1 : 1;
    } else {
      const int hy = tid - nxh, side = hy >= S * bx ? 1 : 0;
      r = side ? hy - S * bx : hy;
      d = r / bx;
      const int xx = r - d * bx;
      f = 2 + side;
      h_at = ((side ? by + d : d - S) + S) * W + kCo + xx;
      in_at = ((side ? by - 1 : 0) + S) * W + kCo + xx;
      in_step = side ? -W : W;
    }
  }
  const int side = f & 1, axis = f >> 1;
  const int nb = fc.nbr[f];
  // distance beyond the face of the neighbour's entry, and inside it of the own one
  const int e_out = side ? d : S - 1 - d, e_in = side ? S - 1 - d : d;
  const bool send = item && !sync && fc.k[f] > 0;
  const bool own = item && fc.own[f] != 0;
  const int cnt = item ? fc.cnt[f] : 0;
  const bool wave_own = __any(own ? 1 : 0);
  int wave_cnt = cnt;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) wave_cnt = max(wave_cnt, __shfl_xor(wave_cnt, o, 64));
  wave_cnt = __builtin_amdgcn_readfirstlane(wave_cnt);
  const bool any_item = __any(item ? 1 : 0);
  // halo source (the synchronous scheme: the neighbour's field)
  const Real* hsrc;
  int64_t hzs;
  {
    const int ly = axis == 1 ? (side ? d : by - S + d) : r / S, lx = axis == 0 ? (side ? d : bx - S + d) : r - d * bx;
    if (sync) {
      hsrc = C + pe_base(nb) + static_cast<int64_t>(item ? ly : 0) * pitch + (item ? lx : 0);
      hzs = zs;
    } else {
      hsrc = F + fc.hbase[f] + r;
      hzs = strip_zs(p, f ^ 1, q.fslots);
    }
  }
  // own entry in the g ring, and the neighbour's points next to the face (for
  // a delay of 0 there): ia = 0, 1, .. from the face
  const Real* gsrc = G + fc.gbase[f] + r;
  const int64_t gzs = strip_zs(p, f, q.anslots);
  Real* gdst = G + fc.pbase[f] + r;
  const int64_t gdzs = strip_zs(p, f ^ 1, q.anslots);
  int64_t n_at, n_step;
  {
    const int lx = axis == 0 ? (side ? 0 : bx - 1) : r - d * bx, ly = axis == 1 ? (side ? 0 : by - 1) : r / S;
    n_at = pe_base(nb) + static_cast<int64_t>(item ? ly : 0) * pitch + (item ? lx : 0);
    // (threads without an item stay on their first point)
    n_step = !item ? 0 : axis == 0 ? (side ? 1 : -1) : (side ? pitch : -pitch);
  }

  struct Ahead {
    R2 c, y0, y1, x0, x1;                  // c, y: plane z + S; x: plane z
    Real h[TT], g[kDrain];
    Real oc[S], oy[S], oy1[M1 ? S : 1];
  };
  auto load_field = [&](Ahead& a, int z) __attribute__((always_inline)) {      // plane z of c and y (in the PE)
    const int64_t o = base + z * zs;
    a.c = ld2<EVEN>(C + o + col, has2);
    a.y0 = ld2<EVEN>(Y0 + o + col, has2);
    if (M1) a.y1 = ld2<EVEN>(Y1 + o + col, has2);
  };
  // everything else of the next plane; the item's sources advance plane by plane
  const Real* hz = hsrc;
  const Real* gz = gsrc;
  int64_t oz = n_at;
  auto load_plane = [&](Ahead& a, int z) __attribute__((always_inline)) {
    const int64_t o = base + z * zs;
    a.x0 = ld2<EVEN>(X0 + o + col, has2);
    a.x1 = ld2<EVEN>(X1 + o + col, has2);
    if (any_item) {
#pragma unroll
      for (int m = 0; m < TT; ++m) a.h[m] = hz[fc.hoff[f][m]];
      if (wave_cnt > 0) {
#pragma unroll
        for (int i = 0; i < kDrain / 2; ++i) a.g[i] = gz[fc.goff[f][i]];
      }
      if (wave_cnt > kDrain / 2) {
#pragma unroll
        for (int i = kDrain / 2; i < kDrain; ++i) a.g[i] = gz[fc.goff[f][i]];
      }
      if (wave_own) {
#pragma unroll
        for (int ia = 0; ia < S; ++ia) {
          const int64_t g = oz + ia * n_step;
          if (BURG) a.oc[ia] = C[g];
          a.oy[ia] = Y0[g];
          if (M1) a.oy1[ia] = Y1[g];
        }
      }
    }
    hz += hzs;
    gz += gzs;
    oz += zs;
  };
  auto taps = [&](int a, int up, int e, const double (&mu)[S], const double (&pr)[S]) __attribute__((always_inline)) {
    return face_taps<S, TT, 6, BURG>(fc, a, up, e, mu, pr);
  };
  const double mf = M1 ? 1.0 : m0;         // factor of the sums over Y values
  auto y_of = [&](Real a, Real b) __attribute__((always_inline)) -> Y {
    if constexpr (M1) return m0 * static_cast<double>(a) + m1 * static_cast<double>(b);
    else return a;
  };

  // ---- z faces: outgoing taps of the first and last S planes, and the c
  // planes beyond the PE (low: registers, high: LDS)
  R2 cq[NT];
  Two<Y> yq[NT];
  const int64_t rz = static_cast<int64_t>(y) * bx + x;
#pragma unroll
  for (int up = 0; up < 2; ++up) {
    const int fz = 4 + up;
    if (active && !sync && fc.k[fz] > 0) {
      double mu[2][S], pr[2][S];
#pragma unroll
      for (int ia = 0; ia < S; ++ia) {
        const int z = up ? bz - 1 - ia : ia;
        const R2 c = ld2<EVEN>(C + base + z * zs + col, has2), a = ld2<EVEN>(Y0 + base + z * zs + col, has2);
        R2 b = a;
        if (M1) b = ld2<EVEN>(Y1 + base + z * zs + col, has2);
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          mu[v][ia] = static_cast<double>(y_of(a.v[v], b.v[v]));
          pr[v][ia] = static_cast<double>(c.v[v]) * mu[v][ia];
        }
      }
#pragma unroll
      for (int e = 0; e < S; ++e) {
        R2 g;
#pragma unroll
        for (int v = 0; v < 2; ++v) g.v[v] = static_cast<Real>(mf * taps(2, up, e, mu[v], pr[v]));
        const int dd = up ? e : S - 1 - e;
        st2<EVEN>(G + fc.pbase[fz] + rz + dd * strip_zs(p, fz ^ 1, q.anslots), g, has2);
      }
    }
#pragma unroll
    for (int dd = 0; dd < S; ++dd) {
      R2 h;
      if (sync) {
        h = ld2<EVEN>(C + pe_base(fc.nbr[fz]) + y * pitch + x + (up ? dd : bz - S + dd) * zs, has2);
      } else {
        const Real* src = F + fc.hbase[fz] + rz + dd * strip_zs(p, fz ^ 1, q.fslots);
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int m = 0; m < TT; ++m) {
          const R2 l = ld2<EVEN>(src + fc.hoff[fz][m], has2);
          s0 += fc.w[fz][m] * static_cast<double>(l.v[0]);
          s1 += fc.w[fz][m] * static_cast<double>(l.v[1]);
        }
        h.v[0] = static_cast<Real>(s0);
        h.v[1] = static_cast<Real>(s1);
      }
      if (up) {
        if (active) st2<EVEN>(sZ + (dd * by + y) * bx + x, h, has2);
      } else {
        cq[dd] = h;
        yq[dd].v[0] = yq[dd].v[1] = Y(0);
      }
    }
  }
  Ahead nx;
#pragma unroll
  for (int i = 0; i < S; ++i) {
    load_field(nx, i);
    cq[S + i] = nx.c;
#pragma unroll
    for (int v = 0; v < 2; ++v) yq[S + i].v[v] = y_of(nx.y0.v[v], M1 ? nx.y1.v[v] : nx.y0.v[v]);
  }
  load_field(nx, S);
  load_plane(nx, 0);

  // constant part of -D: the sum of the first-kind taps (the c1 taps of an
  // axis cancel)
  double ksum = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int o = 1; o <= S; ++o) ksum += fc.t1[a][0][o] + fc.t1[a][1][o];
  // The Laplacian of FP32 fields: a sum of two neighbours rounds at 2^-53 at most
  // (exact while their exponents lie within 29 of each other), far below the
  // fields' own rounding, and the centre enters once (lap0) instead of in every
  // difference: two of the six to eleven FP64 operations of a neighbour pair less.
  // FP64 fields keep the differences, which lose less to cancellation.
  constexpr bool kSum = sizeof(Real) == 4;
  double lap0 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int o = 1; o <= S; ++o) lap0 -= 2.0 * p.c2[a][S + o];

  double da = 0.0;
  for (int z = 0; z < bz; ++z) {
    const int buf = z & 1;
    Real* Cp = sC + buf * plane;
    Y* Yp = sY + buf * plane;
    double* Ap = sA + buf * nh;
    // plane z + S enters the queue
    if (z + S < bz) {
      cq[2 * S] = nx.c;
#pragma unroll
      for (int v = 0; v < 2; ++v) yq[2 * S].v[v] = y_of(nx.y0.v[v], M1 ? nx.y1.v[v] : nx.y0.v[v]);
    } else {
      cq[2 * S] = ld2<EVEN>(sZ + ((z + S - bz) * by + y) * bx + x, has2);
      yq[2 * S].v[0] = yq[2 * S].v[1] = Y(0);
    }
    const R2 xv0 = nx.x0, xv1 = nx.x1;
    if (active) {
      st2<EVEN>(Cp + at, cq[S], has2);
      st2<EVEN>(Yp + at, yq[S], has2);
    }
    if (item) {
      double hs = 0.0;                     // (the synchronous scheme: weights 1, 0, ..)
#pragma unroll
      for (int m = 0; m < TT; ++m) hs += fc.w[f][m] * static_cast<double>(nx.h[m]);
      Cp[h_at] = static_cast<Real>(hs);
      double g = 0.0;
      if (wave_cnt > 0) {
#pragma unroll
        for (int i = 0; i < kDrain / 2; ++i) g += i < cnt ? fc.dw[f][i] * static_cast<double>(nx.g[i]) : 0.0;
      }
      if (wave_cnt > kDrain / 2) {
#pragma unroll
        for (int i = kDrain / 2; i < kDrain; ++i) g += i < cnt ? fc.dw[f][i] * static_cast<double>(nx.g[i]) : 0.0;
        // (gz is a plane ahead)
        for (int i = kDrain; i < cnt; ++i) g += fc.dw[f][i] * static_cast<double>((gz - gzs)[fc.goff[f][i]]);
      }
      if (own) {
        double mu[S], pr[S];
#pragma unroll
        for (int ia = 0; ia < S; ++ia) {
          mu[ia] = m0 * static_cast<double>(nx.oy[ia]) + (M1 ? m1 * static_cast<double>(nx.oy1[M1 ? ia : 0]) : 0.0);
          pr[ia] = BURG ? static_cast<double>(nx.oc[ia]) * mu[ia] : 0.0;
        }
        g += taps(axis, side ^ 1, e_in, mu, pr);
      }
      Ap[tid] = g;
    }
    __syncthreads();
    {
      load_field(nx, z + 1 + S < bz ? z + 1 + S : bz - 1);
      if (z + 1 < bz) load_plane(nx, z + 1);
    }
    if (active) {
      // x row segment and y neighbours of both points
      constexpr int kRow = 2 * (kCo / 2) + 2 + 4;   // columns x - 4 .. x + 5
      Real crow[kRow];
      Y yrow[kRow];
#pragma unroll
      for (int i = 0; i < kRow / 2; ++i) {
        const bool need = 2 * i + 1 >= kCo - S && 2 * i <= kCo + 1 + S;
        if (need) {
          const R2 a = ld2<true>(Cp + at - kCo + 2 * i, true);
          const Two<Y> b = ld2<true>(Yp + at - kCo + 2 * i, true);
          crow[2 * i] = a.v[0];
          crow[2 * i + 1] = a.v[1];
          yrow[2 * i] = b.v[0];
          yrow[2 * i + 1] = b.v[1];
        }
      }
      double acc[2], acc2[2], lap[2], grad[2];   // acc2: to be scaled by alpha (Burgers)
#pragma unroll
      for (int v = 0; v < 2; ++v) acc[v] = acc2[v] = lap[v] = grad[v] = 0.0;
      // a neighbour pair at -o and +o along axis a of point v: the stage field
      // (cm, cp) and mu (ym, yp); a transposed tap from the point at -o has
      // offset +o and the other way round
      auto pair = [&](int a, int o, int v, Real cm_, Real cp_, Y ym_, Y yp_) __attribute__((always_inline)) {
        [[maybe_unused]] const double cj = static_cast<double>(cq[S].v[v]);
        const double cm = static_cast<double>(cm_), cp = static_cast<double>(cp_);
        const double ym = static_cast<double>(ym_), yp = static_cast<double>(yp_);
        if constexpr (kSum) lap[v] += p.c2[a][S + o] * (cm + cp);
        else lap[v] += p.c2[a][S + o] * ((cm - cj) + (cp - cj));
        if constexpr (BURG) {
          grad[v] += p.c1[a][S + o] * (cp - cm);
          acc2[v] += p.c2[a][S + o] * (ym + yp);
          acc[v] -= p.c1[a][S + o] * (cm * ym - cp * yp);
        } else {
          acc[v] += p.kad[a][S + o] * ym;
          acc[v] += p.kad[a][S - o] * yp;
        }
      };
#pragma unroll
      for (int o = 1; o <= S; ++o) {
#pragma unroll
        for (int v = 0; v < 2; ++v)
          pair(0, o, v, crow[kCo + v - o], crow[kCo + v + o], yrow[kCo + v - o], yrow[kCo + v + o]);
        const R2 cm = ld2<true>(Cp + at - o * W, true), cp = ld2<true>(Cp + at + o * W, true);
        const Two<Y> ym = ld2<true>(Yp + at - o * W, true), yp = ld2<true>(Yp + at + o * W, true);
#pragma unroll
        for (int v = 0; v < 2; ++v) pair(1, o, v, cm.v[v], cp.v[v], ym.v[v], yp.v[v]);
#pragma unroll
        for (int v = 0; v < 2; ++v)
          pair(2, o, v, cq[S - o].v[v], cq[S + o].v[v], yq[S - o].v[v], yq[S + o].v[v]);
      }
      double in[2] = {0.0, 0.0};           // drained entries (mu's factor included)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int xv = x + v;
        if (xv < S) in[v] += Ap[y * S + xv];
        if (xv >= bx - S && xv < bx) in[v] += Ap[S * by + y * S + xv - (bx - S)];
        if (xv < bx) {
          if (y < S) in[v] += Ap[nxh + y * bx + xv];
          if (y >= by - S) in[v] += Ap[nxh + S * bx + (y - (by - S)) * bx + xv];
        }
      }
#pragma unroll
      for (int up = 0; up < 2; ++up) {
        if (up ? z < bz - S : z >= S) continue;   // uniform
        const int fz = 4 + up, dd = up ? z - (bz - S) : z, e = up ? S - 1 - dd : dd;
        const Real* src = G + fc.gbase[fz] + rz + dd * strip_zs(p, fz, q.anslots);
        for (int i = 0; i < fc.cnt[fz]; ++i) {
          const R2 g = ld2<EVEN>(src + fc.goff[fz][i], has2);
          in[0] += fc.dw[fz][i] * static_cast<double>(g.v[0]);
          in[1] += fc.dw[fz][i] * static_cast<double>(g.v[1]);
        }
        if (fc.own[fz]) {
          double mu[2][S], pr[2][S];
          const int64_t o0 = pe_base(fc.nbr[fz]) + y * pitch + x;
#pragma unroll
          for (int ia = 0; ia < S; ++ia) {
            const int64_t g = o0 + (up ? ia : bz - 1 - ia) * zs;
            const R2 c = ld2<EVEN>(C + g, has2), a = ld2<EVEN>(Y0 + g, has2);
            R2 b = a;
            if (M1) b = ld2<EVEN>(Y1 + g, has2);
#pragma unroll
            for (int v = 0; v < 2; ++v) {
              mu[v][ia] = m0 * static_cast<double>(a.v[v]) + (M1 ? m1 * static_cast<double>(b.v[v]) : 0.0);
              pr[v][ia] = static_cast<double>(c.v[v]) * mu[v][ia];
            }
          }
#pragma unroll
          for (int v = 0; v < 2; ++v) in[v] += taps(2, up ^ 1, e, mu[v], pr[v]);
        }
      }
      R2 res;
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const double yv = static_cast<double>(yq[S].v[v]);
        const double sum = (BURG ? p.alpha * acc2[v] + acc[v] : acc[v]) - (ksum + (BURG ? grad[v] : 0.0)) * yv;
        res.v[v] = static_cast<Real>(q.b0 * static_cast<double>(xv0.v[v]) + q.b1 * static_cast<double>(xv1.v[v]) +
                                     (mf * sum + in[v]));
        if constexpr (kSum) lap[v] += lap0 * static_cast<double>(cq[S].v[v]);
        if (v == 0 || has2) da += mf * yv * lap[v];
      }
      st2<EVEN>(out + base + z * zs + col, res, has2);
    }
    if (send) {
      double mu[S], pr[S];
#pragma unroll
      for (int ia = 0; ia < S; ++ia) {
        mu[ia] = static_cast<double>(Yp[in_at + ia * in_step]);
        pr[ia] = BURG ? static_cast<double>(Cp[in_at + ia * in_step]) * mu[ia] : 0.0;
      }
      *gdst = static_cast<Real>(mf * taps(axis, side, e_out, mu, pr));
      gdst += gdzs;
    }
#pragma unroll
    for (int i = 0; i < 2 * S; ++i) {
      cq[i] = cq[i + 1];
      yq[i] = yq[i + 1];
    }
  }
  // fixed-order block reduction of the alpha-gradient part
  for (int off = 32; off > 0; off >>= 1) da += __shfl_down(da, off, 64);
  __shared__ double part[MAXT / 64];
  if ((tid & 63) == 0) part[tid / 64] = da;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int w = 0; w < nt / 64; ++w) s += part[w];
    q.partial[pe] += s;
  }
}

template <typename Real, int S, int TT, bool BURG, bool M1, int MAXT>
void launch_even(const AdjParams& q, int threads, size_t lds, hipStream_t st) {
  if (q.sp.bx % 2 == 0)
    hipLaunchKernelGGL((adj3d_kernel<Real, S, TT, BURG, M1, true, MAXT>), dim3(q.sp.npe), dim3(threads), lds, st, q);
  else
    hipLaunchKernelGGL((adj3d_kernel<Real, S, TT, BURG, M1, false, MAXT>), dim3(q.sp.npe), dim3(threads), lds, st, q);
}

template <typename Real, int S, int TT, bool BURG>
void launch_m1(const AdjParams& q, int threads, size_t lds, hipStream_t st) {
  const bool m1 = q.m1 != 0.0;
  if (threads <= 512) {
    if (m1) launch_even<Real, S, TT, BURG, true, 512>(q, threads, lds, st);
    else launch_even<Real, S, TT, BURG, false, 512>(q, threads, lds, st);
  } else {
    if (m1) launch_even<Real, S, TT, BURG, true, 1024>(q, threads, lds, st);
    else launch_even<Real, S, TT, BURG, false, 1024>(q, threads, lds, st);
  }
}

template <typename Real, int S, int TT>
void launch_burg(const AdjParams& q, int threads, size_t lds, hipStream_t st) {
  if (q.burgers) launch_m1<Real, S, TT, true>(q, threads, lds, st);
  else launch_m1<Real, S, TT, false>(q, threads, lds, st);
}

template <typename Real, int S>
void launch_tt(const AdjParams& q, int threads, size_t lds, hipStream_t st) {
  if (q.sp.mode == AT_SYNC || q.sp.T == S + 1) launch_burg<Real, S, S + 1>(q, threads, lds, st);
  else launch_burg<Real, S, kMaxT>(q, threads, lds, st);
}

}  // namespace adj3d

template <typename Real>
hipError_t launch_adj3d(const AdjParams& q, hipStream_t st) {
  using namespace adj3d;
  const StepParams& p = q.sp;
  if (!adj3d_fits(p, sizeof(Real) == 8) || p.bz < 2 * p.s || q.anslots < 1) return hipErrorInvalidValue;
  const int threads = adj3d_threads(p);
  const size_t lds = adj3d_lds(p, sizeof(Real), q.m1 != 0.0);
  switch (p.s) {
    case 1: launch_tt<Real, 1>(q, threads, lds, st); break;
    case 2: launch_tt<Real, 2>(q, threads, lds, st); break;
    case 3: launch_tt<Real, 3>(q, threads, lds, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace atfd
