// Stage of the reversed step for 1-D and 2-D problems: one workgroup per PE,
// the PE's plane in LDS (adjoint_gather.hpp: how the strips are done).
//
// What bounds it: latency, then FP64 issue. The plane is read and computed once,
// so a stage is the launch, one round of loads (the plane's own values, issued
// before the delays are drawn), one round of strip loads, the arithmetic (about
// 45 FP64 instructions a point, two fifths of the time) and the stores; two
// barriers besides that of the face set-up. 1024^2 in 16^2 PEs, fourth-order
// AB2, FP32: 11.2 us a stage; 14.1 us while parameters were read at run-time
// addresses and every drained value had its own wait; 25 us with a scatter that
// read and wrote back T ring slots per strip value before the plane could be used.
#pragma once

#include "adjoint_gather.hpp"

namespace atfd {
namespace adj2d {

using namespace adjg;

constexpr int kPre = 2;          // pairs of points a thread loads before the set-up

template <typename Real, int DIM, int S, int TT, bool BURG, bool M1, bool EVEN>
__global__ __launch_bounds__(1024) void adj2d_kernel(AdjParams q) {
  const StepParams& p = q.sp;
  using Y = typename std::conditional<M1, double, Real>::type;   // mu (M1), or y0 with m0 applied at the end
  using R2 = Two<Real>;
  constexpr int NF = 2 * DIM;
  constexpr int kCo = 4;                   // LDS column of x = 0
  constexpr int SY = DIM == 2 ? S : 0;     // frame rows
  extern __shared__ __align__(16) unsigned char smem[];
  const int bx = p.bx, by = DIM == 2 ? p.by : 1;
  const int W = (bx + kCo + S + 2) & ~1, H = by + 2 * SY;
  const int plane = W * H;
  const int nxh = 2 * S * by, nh = nxh + (DIM == 2 ? 2 * S * bx : 0);
  double* sA = reinterpret_cast<double*>(smem);              // [nh] drained entries
  Y* sY = reinterpret_cast<Y*>(sA + nh);                     // [plane]
  Real* sC = reinterpret_cast<Real*>(sY + plane);            // [plane]
  __shared__ Faces<S, TT, NF> fc;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int pe = blockIdx.x;
  const int64_t n = q.n;
  const bool sync = p.mode == AT_SYNC;
  const double m0 = q.m0, m1 = q.m1;
  const int qy = div_index(pe, p.px), qx = pe - qy * p.px;
  const int64_t pitch = p.nx;
  auto pe_base = [&](int e) __attribute__((always_inline)) -> int64_t {
    const int ey = div_index(e, p.px), ex = e - ey * p.px;
    return static_cast<int64_t>(ey) * by * pitch + static_cast<int64_t>(ex) * bx;
  };
  const int64_t base = static_cast<int64_t>(qy) * by * pitch + static_cast<int64_t>(qx) * bx;
  const Real* __restrict__ C = static_cast<const Real*>(q.levels) + (n - q.seg_start) * q.npts;
  const Real* __restrict__ Y0 = static_cast<const Real*>(q.y0);
  const Real* __restrict__ Y1 = static_cast<const Real*>(M1 ? q.y1 : q.y0);
  const Real* __restrict__ X0 = static_cast<const Real*>(q.x0);
  const bool b1 = q.b1 != 0.0;
  const Real* __restrict__ X1 = static_cast<const Real*>(b1 ? q.x1 : q.x0);
  Real* __restrict__ out = static_cast<Real*>(q.out);
  const Real* __restrict__ F = static_cast<const Real*>(q.fring);
  Real* G = static_cast<Real*>(q.aring);
  const double mf = M1 ? 1.0 : m0;         // factor of the sums over Y values
  auto y_of = [&](Real a, Real b) __attribute__((always_inline)) -> Y {
    if constexpr (M1) return m0 * static_cast<double>(a) + m1 * static_cast<double>(b);
    else return a;
  };

  // ---- the plane's own values: a thread's first kPre pairs of points are in
  // flight while the delays are drawn
  const int vx = (bx + 1) / 2, nvec = vx * by;
  struct Own {
    R2 c, y0, y1, x0, x1;
  };
  auto load_own = [&](Own& o, int i) __attribute__((always_inline)) {
    const int y = DIM == 2 ? div_small(i, vx) : 0, x = 2 * (i - y * vx);
    const bool has2 = EVEN || x + 1 < bx;
    const int64_t g = base + y * pitch + x;
    o.c = ld2<EVEN>(C + g, has2);
    o.y0 = ld2<EVEN>(Y0 + g, has2);
    if (M1) o.y1 = ld2<EVEN>(Y1 + g, has2);
    o.x0 = ld2<EVEN>(X0 + g, has2);
    o.x1 = ld2<EVEN>(X1 + g, has2);
  };
  auto put_own = [&](const Own& o, int i) __attribute__((always_inline)) {
    const int y = DIM == 2 ? div_small(i, vx) : 0, x = 2 * (i - y * vx);
    const bool has2 = EVEN || x + 1 < bx;
    const int at = (y + SY) * W + kCo + x;
    Two<Y> m;
#pragma unroll
    for (int v = 0; v < 2; ++v) m.v[v] = y_of(o.y0.v[v], M1 ? o.y1.v[v] : o.y0.v[v]);
    st2<EVEN>(sC + at, o.c, has2);
    st2<EVEN>(sY + at, m, has2);
  };
  Own pre[kPre];
#pragma unroll
  for (int k = 0; k < kPre; ++k) load_own(pre[k], tid + k * nt < nvec ? tid + k * nt : 0);
  const double part0 = __hip_atomic_load(&q.partial[pe], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // zero frame of mu
  for (int i = tid; i < plane; i += nt) sY[i] = Y(0);
  face_setup<S, TT, NF, BURG>(q, pe, fc);

  // ---- items of the x / y frame: side and depth d of a face's strip, line.
  // Beyond the face: the neighbour's strip, entry r (halo value in, outgoing
  // taps out); inside it: this PE's own strip, entry r.
  struct Item {
    int f, r, d, line;
  };
  auto item_of = [&](int h) __attribute__((always_inline)) {
    Item t;
    if (h < nxh) {
      const int side = h >= S * by ? 1 : 0;
      t.f = side;
      t.r = side ? h - S * by : h;
      t.line = t.r / S;
      t.d = t.r - t.line * S;
    } else {
      const int hy = h - nxh, side = hy >= S * bx ? 1 : 0;
      t.f = 2 + side;
      t.r = side ? hy - S * bx : hy;
      t.d = div_small(t.r, bx);
      t.line = t.r - t.d * bx;
    }
    return t;
  };
  for (int h = tid; h < nh; h += nt) {
    const Item t = item_of(h);
    const int side = t.f & 1, axis = t.f >> 1, nb = fc.nbr[t.f];
    // halo value of the stage field
    const Real* hsrc;
    if (sync) {
      const int a = side ? t.d : (axis ? by : bx) - S + t.d;
      hsrc = C + pe_base(nb) + (axis ? a * pitch + t.line : t.line * pitch + a);
    } else {
      hsrc = F + fc.hbase[t.f] + t.r;
    }
    Real hv[TT];
#pragma unroll
    for (int m = 0; m < TT; ++m) hv[m] = hsrc[fc.hoff[t.f][m]];
    // entries of the g ring that reach level n
    // (the synchronous scheme has none: any value, dropped below)
    const Real* gsrc = sync ? hsrc : G + fc.gbase[t.f] + t.r;
    const int cnt = fc.cnt[t.f];
    Real gv[kDrain];
#pragma unroll
    for (int i = 0; i < kDrain; ++i) gv[i] = gsrc[fc.goff[t.f][i]];
    // the neighbour's points next to the face, where its delay is 0
    const bool own = fc.own[t.f] != 0;
    Real oc[S], oy[S], oy1[M1 ? S : 1];
    if (own) {
      const int64_t o0 = pe_base(nb) + (axis ? (side ? 0 : by - 1) * pitch + t.line
                                             : t.line * pitch + (side ? 0 : bx - 1));
      const int64_t step = (side ? 1 : -1) * (axis ? pitch : 1);
#pragma unroll
      for (int ia = 0; ia < S; ++ia) {
        if (BURG) oc[ia] = C[o0 + ia * step];
        oy[ia] = Y0[o0 + ia * step];
        if (M1) oy1[ia] = Y1[o0 + ia * step];
      }
    }
    double hs = 0.0;                       // (the synchronous scheme: weights 1, 0, ..)
#pragma unroll
    for (int m = 0; m < TT; ++m) hs += fc.w[t.f][m] * static_cast<double>(hv[m]);
    const int out_at = side ? (axis ? by : bx) + t.d : t.d - S;
    sC[axis ? (out_at + SY) * W + kCo + t.line : (t.line + SY) * W + kCo + out_at] = static_cast<Real>(hs);
    double g = 0.0;
#pragma unroll
    for (int i = 0; i < kDrain; ++i) g += i < cnt ? fc.dw[t.f][i] * static_cast<double>(gv[i]) : 0.0;
    for (int i = kDrain; i < cnt; ++i) g += fc.dw[t.f][i] * static_cast<double>(gsrc[fc.goff[t.f][i]]);
    if (own) {
      double mu[S], pr[S];
#pragma unroll
      for (int ia = 0; ia < S; ++ia) {
        mu[ia] = m0 * static_cast<double>(oy[ia]) + (M1 ? m1 * static_cast<double>(oy1[M1 ? ia : 0]) : 0.0);
        pr[ia] = BURG ? static_cast<double>(oc[ia]) * mu[ia] : 0.0;
      }
      g += face_taps<S, TT, NF, BURG>(fc, axis, side ^ 1, side ? S - 1 - t.d : t.d, mu, pr);
    }
    sA[h] = g;
  }
#pragma unroll
  for (int k = 0; k < kPre; ++k)
    if (tid + k * nt < nvec) put_own(pre[k], tid + k * nt);
  for (int i = tid + kPre * nt; i < nvec; i += nt) {
    Own o;
    load_own(o, i);
    put_own(o, i);
  }
  __syncthreads();

  // ---- transposed taps that leave the PE across a face with a delay
  if (!sync)
    for (int h = tid; h < nh; h += nt) {
      const Item t = item_of(h);
      if (fc.k[t.f] == 0) continue;
      const int side = t.f & 1, axis = t.f >> 1;
      const int in_at = axis ? ((side ? by - 1 : 0) + SY) * W + kCo + t.line : (t.line + SY) * W + kCo + (side ? bx - 1 : 0);
      const int step = (side ? -1 : 1) * (axis ? W : 1);
      double mu[S], pr[S];
#pragma unroll
      for (int ia = 0; ia < S; ++ia) {
        mu[ia] = static_cast<double>(sY[in_at + ia * step]);
        pr[ia] = BURG ? static_cast<double>(sC[in_at + ia * step]) * mu[ia] : 0.0;
      }
      G[fc.pbase[t.f] + t.r] =
          static_cast<Real>(mf * face_taps<S, TT, NF, BURG>(fc, axis, side, side ? t.d : S - 1 - t.d, mu, pr));
    }

  // ---- the points. Constant part of -D: the sum of the first-kind taps (the
  // c1 taps of an axis cancel)
  double ksum = 0.0;
#pragma unroll
  for (int a = 0; a < DIM; ++a)
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
  for (int a = 0; a < DIM; ++a)
#pragma unroll
    for (int o = 1; o <= S; ++o) lap0 -= 2.0 * p.c2[a][S + o];
  double da = 0.0;
  auto points = [&](int i, const R2& x0, const R2& x1) __attribute__((always_inline)) {
    const int y = DIM == 2 ? div_small(i, vx) : 0, x = 2 * (i - y * vx);
    const bool has2 = EVEN || x + 1 < bx;
    const int at = (y + SY) * W + kCo + x;
    constexpr int kRow = kCo + 6;          // columns x - 4 .. x + 5
    Real crow[kRow];
    Y yrow[kRow];
#pragma unroll
    for (int j = 0; j < kRow / 2; ++j) {
      if (2 * j + 1 >= kCo - S && 2 * j <= kCo + 1 + S) {
        const R2 a = ld2<true>(sC + at - kCo + 2 * j, true);
        const Two<Y> b = ld2<true>(sY + at - kCo + 2 * j, true);
        crow[2 * j] = a.v[0];
        crow[2 * j + 1] = a.v[1];
        yrow[2 * j] = b.v[0];
        yrow[2 * j + 1] = b.v[1];
      }
    }
    // acc2: to be scaled by alpha (Burgers)
    double acc[2] = {0.0, 0.0}, acc2[2] = {0.0, 0.0}, lap[2] = {0.0, 0.0}, grad[2] = {0.0, 0.0};
    // a neighbour pair at -o and +o along axis a of point v: the stage field
    // (cm, cp) and mu (ym, yp); a transposed tap from the point at -o has
    // offset +o and the other way round
    auto pair = [&](int a, int o, int v, Real cm_, Real cp_, Y ym_, Y yp_) __attribute__((always_inline)) {
      [[maybe_unused]] const double cj = static_cast<double>(crow[kCo + v]);
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
      if constexpr (DIM == 2) {
        const R2 cm = ld2<true>(sC + at - o * W, true), cp = ld2<true>(sC + at + o * W, true);
        const Two<Y> ym = ld2<true>(sY + at - o * W, true), yp = ld2<true>(sY + at + o * W, true);
#pragma unroll
        for (int v = 0; v < 2; ++v) pair(1, o, v, cm.v[v], cp.v[v], ym.v[v], yp.v[v]);
      }
    }
    R2 res;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int xv = x + v;
      double in = 0.0;                     // drained entries (mu's factor included)
      if (xv < S) in += sA[y * S + xv];
      if (xv >= bx - S && xv < bx) in += sA[S * by + y * S + xv - (bx - S)];
      if (DIM == 2 && xv < bx) {
        if (y < S) in += sA[nxh + y * bx + xv];
        if (y >= by - S) in += sA[nxh + S * bx + (y - (by - S)) * bx + xv];
      }
      const double yv = static_cast<double>(yrow[kCo + v]);
      const double sum = (BURG ? p.alpha * acc2[v] + acc[v] : acc[v]) - (ksum + (BURG ? grad[v] : 0.0)) * yv;
      res.v[v] = static_cast<Real>(q.b0 * static_cast<double>(x0.v[v]) + q.b1 * static_cast<double>(x1.v[v]) +
                                   (mf * sum + in));
      if constexpr (kSum) lap[v] += lap0 * static_cast<double>(crow[kCo + v]);
      if (v == 0 || has2) da += mf * yv * lap[v];
    }
    st2<EVEN>(out + base + y * pitch + x, res, has2);
  };
#pragma unroll
  for (int k = 0; k < kPre; ++k)
    if (tid + k * nt < nvec) points(tid + k * nt, pre[k].x0, pre[k].x1);
  for (int i = tid + kPre * nt; i < nvec; i += nt) {
    const int y = DIM == 2 ? div_small(i, vx) : 0, x = 2 * (i - y * vx);
    const bool has2 = EVEN || x + 1 < bx;
    const int64_t g = base + y * pitch + x;
    points(i, ld2<EVEN>(X0 + g, has2), ld2<EVEN>(X1 + g, has2));
  }

  // fixed-order block reduction of the alpha-gradient part
  for (int off = 32; off > 0; off >>= 1) da += __shfl_down(da, off, 64);
  __shared__ double part[1024 / 64];
  if ((tid & 63) == 0) part[tid / 64] = da;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int w = 0; w < nt / 64; ++w) s += part[w];
    q.partial[pe] = part0 + s;
  }
}

template <typename Real, int DIM, int S, int TT, bool BURG>
void launch_form(const AdjParams& q, int threads, size_t lds, hipStream_t st) {
  const bool m1 = q.m1 != 0.0, even = q.sp.bx % 2 == 0;
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(q.sp.npe), dim3(threads), lds, st, q); };
  if (m1 && even) go(adj2d_kernel<Real, DIM, S, TT, BURG, true, true>);
  else if (m1) go(adj2d_kernel<Real, DIM, S, TT, BURG, true, false>);
  else if (even) go(adj2d_kernel<Real, DIM, S, TT, BURG, false, true>);
  else go(adj2d_kernel<Real, DIM, S, TT, BURG, false, false>);
}

template <typename Real, int DIM, int S>
void launch_tt(const AdjParams& q, int threads, size_t lds, hipStream_t st) {
  if (q.sp.mode == AT_SYNC || q.sp.T == S + 1) {
    if (q.burgers) launch_form<Real, DIM, S, S + 1, true>(q, threads, lds, st);
    else launch_form<Real, DIM, S, S + 1, false>(q, threads, lds, st);
  } else {
    if (q.burgers) launch_form<Real, DIM, S, kMaxT, true>(q, threads, lds, st);
    else launch_form<Real, DIM, S, kMaxT, false>(q, threads, lds, st);
  }
}

}  // namespace adj2d

template <typename Real, int DIM>
hipError_t launch_adj2d(const AdjParams& q, hipStream_t st) {
  using namespace adj2d;
  const StepParams& p = q.sp;
  if (p.ndim != DIM || !adj2d_applies(p, sizeof(Real) == 8) || q.anslots < 1) return hipErrorInvalidValue;
  const int threads = adj2d_threads(p);
  const size_t lds = adj2d_lds(p, sizeof(Real), q.m1 != 0.0);
  switch (p.s) {
    case 1: launch_tt<Real, DIM, 1>(q, threads, lds, st); break;
    case 2: launch_tt<Real, DIM, 2>(q, threads, lds, st); break;
    case 3: launch_tt<Real, DIM, 3>(q, threads, lds, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace atfd
