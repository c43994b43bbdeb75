// Degrees past the compile-time kernels (float l_max > 12, double > 8): one
// lane per (point, order).
//
// A row of harmonics no longer fits a 16-point LDS tile there, and the tile
// is what makes the stores contiguous: so a block takes few points (P, see
// ord_shape) and finds its parallelism in the orders instead.  Thread i of
// the block owns order m = i / P of point i % P and walks the degrees
// l = m .. l_max upward at fixed order, with a few values of state instead of
// a row (OrdChain).  All lanes of a wave are at the same l: the lanes of one
// point write neighbouring columns of the LDS tile, and the coefficients of a
// degree are one contiguous read.  A wave starts at its lowest order, so the
// waves of high orders are short.
//
// The tile is laid out like global memory ([P] rows of Y, then [P][3] rows of
// dY, each block shifted so that it is congruent to its global address modulo
// 16 bytes) and leaves as 16-byte stores whatever the alignment.
#pragma once

#include "sph_device.hpp"
#include "sph_fwd.inl"
#include "sph_launch.hpp"

namespace sph {

constexpr int kOrdThreads = 512;  // most threads of a block

// LDS of one k_ord block: the tile's Y, dY and gY (each of whole 16-byte
// vectors, one more for its shift) and the backward's sums per order.
template <typename T>
__host__ __device__ constexpr int ord_block(int elems) {
  constexpr int W = 16 / static_cast<int>(sizeof(T));
  return (elems + W - 1) / W * W + W;
}
template <typename T>
__host__ __device__ constexpr size_t ord_lds_bytes(int L, int points, bool store_y, bool store_dy, bool bwd) {
  const int K = (L + 1) * (L + 1);
  return sizeof(T) * ((store_y ? static_cast<size_t>(ord_block<T>(points * K)) : 0) +
                      (store_dy ? static_cast<size_t>(ord_block<T>(3 * points * K)) : 0) +
                      (bwd ? static_cast<size_t>(ord_block<T>(points * K)) + 3u * (L + 1) * points : 0));
}

// Points per k_ord tile and whether its (point, order) pairs are split
// between two sets of waves.
//   Values or the backward alone: a short pass per tile, for which full
//   waves count.  The most points whose orders fill two waves, or three or
//   one where they are fuller by 7 % (float, values: l_max 32 4.5 TB/s with 5
//   points, 4.2 with 3; l_max 24 4.5 with 5, 4.3 with 7), with at least four
//   blocks in a CU's LDS (double l_max 32: 4.5 TB/s with 3 points, 4.2 with
//   5).
//   Derivatives: a point's four rows decide how many blocks a CU's LDS
//   holds.  Up to 12 KiB per point: as many points as leave four blocks
//   (float l_max 13 5.3 TB/s with 13 points, 4.4 with 4; l_max 16 5.0 with 8,
//   4.3 with 16; double l_max 9 5.8 with 12, 5.2 with 4).  Beyond, where
//   that is one or two waves each: three blocks, and the split, which
//   doubles the waves on the same LDS (float l_max 32, 3 points: 4.25 TB/s,
//   3.8 without; double l_max 32, 2 points: 3.6 and 2.9; but float l_max 13
//   4.5 and 4.6, l_max 20 4.2 and 4.6).
struct OrdShape {
  int points;
  bool split;
};
template <typename T>
constexpr OrdShape ord_shape(int L, bool store_y, bool store_dy, bool bwd) {
  auto lds = [&](int p) { return ord_lds_bytes<T>(L, p, store_y, store_dy, bwd); };
  const int most = kOrdThreads / (L + 1) < 16 ? kOrdThreads / (L + 1) : 16;
  if (store_dy) {
    const bool split = 4 * sizeof(T) * (L + 1) * (L + 1) > 12 * 1024;
    int p = split ? (most < 7 ? most : 7) : most;  // the split's two halves stay within one block's threads
    while (p > 2 && lds(p) > (split ? 53760u : 41984u)) --p;
    return OrdShape{p, split};
  }
  auto pw = [&](int w) { return 64 * w / (L + 1) < most ? 64 * w / (L + 1) : most; };
  auto fill = [&](int w) { return 100 * pw(w) * (L + 1) / (64 * w); };  // percent of the lanes
  int w = 2;
  if (fill(3) >= fill(2) + 7) w = 3;
  if (fill(1) >= fill(w) + 7) w = 1;
  while (w > 1 && lds(pw(w)) > 40 * 1024) --w;
  return OrdShape{pw(w), false};
}

// Two coefficients per (l, m), m <= l (0 elsewhere), read together: N_l^m and
// 1 / (l+m), see OrdChain; rows past kMaxL for the loads ahead of the last
// degree.
constexpr int kOrdStep = 4;  // degrees per trip of the loop over l
template <typename T>
struct OrdTable {
  T a[kMaxL + 1 + 2 * kOrdStep][2 * (kMaxL + 2)];
};

template <typename T>
constexpr OrdTable<T> make_ord_table(int conv) {
  OrdTable<T> t{};
  for (int m = 0; m <= kMaxL; ++m) {
    // N_m^m = Qt_m^m, N_l / N_{l-1} = sqrt((2l+1)/(2l-1) (l+m)/(l-m))
    double n = csqrt(1.0 / (2.0 * kPi));
    for (int j = 1; j <= m; ++j) n *= csqrt(double(2 * j + 1) / double(2 * j));
    for (int l = m; l <= kMaxL; ++l) {
      if (l > m) n *= csqrt(double(2 * l + 1) / double(2 * l - 1) * (double(l + m) / double(l - m)));
      t.a[l][2 * m] = static_cast<T>(n * conv_factor(conv, l));
      t.a[l][2 * m + 1] = l + m > 0 ? static_cast<T>(1.0 / double(l + m)) : T(0);
    }
  }
  return t;
}

// One table per set of factors: this library's (and e3nn's "integral"),
// "component", "norm".
template <typename T>
struct OrdTables {
  OrdTable<T> t[3];
};
constexpr OrdTables<float> kOrdF = {{make_ord_table<float>(0), make_ord_table<float>(2), make_ord_table<float>(3)}};
constexpr OrdTables<double> kOrdD = {{make_ord_table<double>(0), make_ord_table<double>(2), make_ord_table<double>(3)}};

template <typename T>
__device__ __forceinline__ const OrdTable<T>& ord_table(int conv) {
  const int i = conv < 2 ? 0 : conv - 1;
  if constexpr (sizeof(T) == 4)
    return kOrdF.t[i];
  else
    return kOrdD.t[i];
}

// The arithmetic below names its fused operations instead of leaving them to
// the compiler, whose choice depends on which outputs a kernel has: every
// k_ord gives the same bits for the same point.
__device__ __forceinline__ float ord_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double ord_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The recursion upward in l at fixed order m, on the polynomials relative to
// their value on the polar axis, p_l = Qt_l^m / N_l^m (z^(l-m) there).  The
// three-term relation of the solid Ferrers functions,
//   (l+m) p_l = (2l-1) z p_{l-1} - (l-1-m) (z^2 + rho^2) p_{l-2},
// is carried through d_l = p_l - z p_{l-1}:
//   d_l = a (z d_{l-1} - rho^2 p_{l-2}),  p_l = z p_{l-1} + d_l,
//   a = (l-1-m) / (l+m)
// so that, as in the recursion downward in m, the polar angle enters through
// z and rho^2 separately and errors next to the poles do not grow faster than
// the harmonics do (the relation in z and r^2 loses l^2 there).  The
// derivative along x is x E, along y y E, with E = N e, e = 2 dp/d(rho^2):
//   f_l = a (z f_{l-1} - rho^2 e_{l-2} - 2 p_{l-2}),  e_l = z e_{l-1} + f_l
// and the derivative along z is Z = N_l^m (l-m) p_{l-1}.  It starts at l = m:
// lanes of a higher order than the wave's degree wait.
template <typename T>
struct OrdChain {
  T z, rho2;
  T x = T(0);  // l - m
  T p = T(1), pl = T(0), d = T(0);
  T e = T(0), el = T(0), f = T(0);
  // 1 / (l + m) of the next degree
  template <bool XY>
  __device__ __forceinline__ void advance(T inv) {
#pragma clang fp contract(off)
    const T a = x * inv;  // (l' - 1 - m) / (l' + m) at l' = l + 1
    if constexpr (XY) {
      f = a * ord_fma(z, f, -ord_fma(rho2, el, pl + pl));
      el = e;
      e = ord_fma(z, e, f);
    }
    d = a * ord_fma(z, d, -(rho2 * pl));
    pl = p;
    p = ord_fma(z, p, d);
    x += T(1);
  }
};

// The products of the second derivatives: as they are, and with 0 times
// anything 0.
struct MulPlain {
  template <typename T>
  __device__ __forceinline__ T operator()(T a, T b) const {
    return a * b;
  }
};
struct MulZero {
  template <typename T>
  __device__ __forceinline__ T operator()(T a, T b) const {
    // one comparison of both, that is none of a loop-invariant factor alone
    // (kept from trip to trip those spill scalar registers)
    return fmin(fabs(a), fabs(b)) == T(0) ? T(0) : a * b;
  }
};

// OrdChain's recursion carried one derivative further, w = 2 de/d(rho^2):
//   g_l = a (z g_{l-1} - rho^2 w_{l-2} - 4 e_{l-2}),  w_l = z w_{l-1} + g_l.
// p1, e1, w1 and p2: one and two degrees below.  Scaled harmonics far from the
// origin (past reach2 of the launch's parameters) have values past the type's
// range beside derivatives within it, and rho^2 itself may be: there mul is
// MulZero, so that what the degree does not reach yet stays 0.
template <typename T>
struct HessChain {
  T z, rho2;
  T x = T(0);  // l - m
  T p = T(1), p1 = T(0), p2 = T(0), d = T(0);
  T e = T(0), e1 = T(0), f = T(0);
  T w = T(0), w1 = T(0), g = T(0);
  // inv: 1 / (l + m) of the next degree
  template <typename Mul>
  __device__ __forceinline__ void advance(T inv, Mul mul) {
    const T a = x * inv;
    g = mul(a, mul(z, g) - (mul(rho2, w1) + T(4) * e1));
    w1 = w;
    w = mul(z, w) + g;
    f = mul(a, mul(z, f) - (mul(rho2, e1) + T(2) * p1));
    e1 = e;
    e = mul(z, e) + f;
    d = mul(a, mul(z, d) - mul(rho2, p1));
    p2 = p1;
    p1 = p;
    p = mul(z, p) + d;
    x += T(1);
  }
};

// cnt elements between LDS st[shift + j] and global g[j], where shift is g's
// element offset from a 16-byte boundary: the aligned middle as 16-byte
// accesses, a batch of them in flight per thread, the ends one by one.
constexpr int kOrdBatch = 8;

template <typename T>
__device__ __forceinline__ int ord_shift(const T* g) {
  return static_cast<int>((reinterpret_cast<uintptr_t>(g) / sizeof(T)) % Vec16<T>::n);
}

template <typename T>
__device__ __forceinline__ void ord_copy_out(const T* st, int shift, T* g, int cnt, int tid, int nt) {
  using V = typename Vec16<T>::type;
  constexpr int W = Vec16<T>::n;
  int head = (W - shift) % W;
  head = head < cnt ? head : cnt;
  const int nv = (cnt - head) / W;
  const V* sv = reinterpret_cast<const V*>(st + shift + head);
  V* gv = reinterpret_cast<V*>(g + head);
  // vectors [v0, v1) fill whole 128-byte lines and leave with the streaming
  // policy; the line parts at both ends, which neighbouring tiles complete,
  // leave with the default one, so that L2 merges them
  constexpr int kLine = 128 / 16;
  int v0 = (kLine - static_cast<int>((reinterpret_cast<uintptr_t>(gv) / 16) % kLine)) % kLine;
  v0 = v0 < nv ? v0 : nv;
  const int v1 = v0 + (nv - v0) / kLine * kLine;
  const __amdgpu_buffer_rsrc_t rs = stream_rsrc(g + head, nv * 16);
  for (int i0 = v0 + tid; i0 < v1; i0 += nt * kOrdBatch) {
    V v[kOrdBatch];
#pragma unroll
    for (int u = 0; u < kOrdBatch; ++u)
      if (i0 + u * nt < v1) v[u] = sv[i0 + u * nt];
#pragma unroll
    for (int u = 0; u < kOrdBatch; ++u)
      if (i0 + u * nt < v1) stream_store16(v[u], rs, (i0 + u * nt) * 16);
  }
  if (tid < v0) gv[tid] = sv[tid];
  if (tid < nv - v1) gv[v1 + tid] = sv[v1 + tid];
  if (tid < head) g[tid] = st[shift + tid];
  const int t0 = head + nv * W;
  if (tid < cnt - t0) g[t0 + tid] = st[shift + t0 + tid];
}

template <typename T>
__device__ __forceinline__ void ord_copy_in(T* st, int shift, const T* g, int cnt, int tid, int nt) {
  using V = typename Vec16<T>::type;
  constexpr int W = Vec16<T>::n;
  int head = (W - shift) % W;
  head = head < cnt ? head : cnt;
  const int nv = (cnt - head) / W;
  V* sv = reinterpret_cast<V*>(st + shift + head);
  const V* gv = reinterpret_cast<const V*>(g + head);
  for (int i0 = tid; i0 < nv; i0 += nt * kOrdBatch) {
    V v[kOrdBatch];
#pragma unroll
    for (int u = 0; u < kOrdBatch; ++u)
      if (i0 + u * nt < nv) v[u] = __builtin_nontemporal_load(gv + i0 + u * nt);
#pragma unroll
    for (int u = 0; u < kOrdBatch; ++u)
      if (i0 + u * nt < nv) sv[i0 + u * nt] = v[u];
  }
  if (tid < head) st[shift + tid] = g[tid];
  const int t0 = head + nv * W;
  if (tid < cnt - t0) st[shift + t0 + tid] = g[t0 + tid];
}

// SY, SD: Y, dY are stored; BWD: grad_xyz from P.gY.  P.tile points per
// block, (L + 1) P.tile threads rounded up to whole waves.  Dynamic LDS:
// ord_lds_bytes.  A grid-stride loop over tiles, so any grid is correct.
// SPLIT: two threads per (point, order), in waves of their own: the first
// half of the block forms the values and z derivatives, the second the x and
// y derivatives, each with its own recursion.
template <typename T, bool NORM, bool SY, bool SD, bool BWD, bool SPLIT>
__global__ __launch_bounds__(kOrdThreads) void k_ord(FwdParams P) {
#pragma clang fp contract(off)
  constexpr T kIS2 = T(kInvSqrt2d);
  extern __shared__ __align__(16) unsigned char smem[];
  const int L = P.L;
  const int K = (L + 1) * (L + 1);
  const int PT = P.tile;
  const int tid = threadIdx.x, nt = blockDim.x;
  // LDS blocks, each of a whole number of 16-byte vectors plus one
  const int by = ord_block<T>(PT * K), bd = ord_block<T>(3 * PT * K);
  T* sy = reinterpret_cast<T*>(smem);
  T* sd = sy + (SY ? by : 0);
  T* sg = sd + (SD ? bd : 0);
  T* sacc = sg + (BWD ? by : 0);

  if (P.status != nullptr && blockIdx.x == 0 && tid < kWave) check_offsets(P, tid);

  const OrdTable<T>& C = ord_table<T>(P.conv);
  const int half = SPLIT ? nt / 2 : nt;  // whole waves
  const int part = SPLIT ? __builtin_amdgcn_readfirstlane(tid / half) : 0;
  const int it = tid - part * half;  // (order, point) of this thread
  const int m = it / PT, p = it - m * PT;
  const bool lane_on = m <= L;
  const int mm = lane_on ? m : L;
  // the wave's lowest order (past l_max: a wave without one, whose loop is empty)
  const int lw = __builtin_amdgcn_readfirstlane(it / kWave * kWave / PT);
  const int l0 = lw <= L ? lw : L + 1;
  const int64_t tiles = (P.n + PT - 1) / PT;
  for (int64_t tile = xcd_slot(blockIdx.x, gridDim.x); tile < tiles; tile += gridDim.x) {
    const int64_t p0 = tile * PT;
    const int np = static_cast<int>(P.n - p0 < PT ? P.n - p0 : PT);
    const T* xp = static_cast<const T*>(P.xyz) + (p0 + (p < np ? p : np - 1)) * 3;
    const Point<T> pt = make_point<T, NORM>(xp[0], xp[1], xp[2]);
    T* gy = SY ? static_cast<T*>(P.Y) + p0 * K : nullptr;
    T* gd = SD ? static_cast<T*>(P.dY) + p0 * 3 * K : nullptr;
    const T* gg = BWD ? static_cast<const T*>(P.gY) + p0 * K : nullptr;
    const int hy = SY ? ord_shift(gy) : 0, hd = SD ? ord_shift(gd) : 0, hg = BWD ? ord_shift(gg) : 0;
    if constexpr (BWD) {
      ord_copy_in(sg, hg, gg, np * K, tid, nt);
      __syncthreads();
    }
    // The evaluation point and its powers in double: rounding errors of
    // (x + i y)^m grow with m, and the few dozen operations are once per
    // (point, order).
    double ux = xp[0], uy = xp[1], uz = xp[2], ui = 1.0;
    if constexpr (NORM) {
      // one Newton step on the kernel's own 1/r (0 at the origin)
      ui = static_cast<double>(pt.inv_r);
      if constexpr (!std::is_same_v<T, double>) {
        const double rr = ux * ux + uy * uy + uz * uz;
        ui = pt.inv_r == T(0) ? 0.0 : ui * (1.5 - 0.5 * rr * ui * ui);
      }
      ux *= ui;
      uy *= ui;
      uz *= ui;
    }
    // (x + i y)^(m-1) by squaring, then one more factor: c_m, s_m
    double c1 = 1.0, s1 = 0.0;
    {
      double bc = ux, bs = uy;
#pragma unroll
      for (int b = 0; b < 5; ++b) {
        if (((mm - 1) >> b) & 1) {
          const double t = c1 * bc - s1 * bs;
          s1 = c1 * bs + s1 * bc;
          c1 = t;
        }
        const double t = bc * bc - bs * bs;
        bs = 2.0 * bc * bs;
        bc = t;
      }
    }
    T c = static_cast<T>(c1 * ux - s1 * uy), s = static_cast<T>(c1 * uy + s1 * ux);
    // derivative factors, with the normalised derivatives' 1/r folded in
    T mc = static_cast<T>(mm * c1 * ui), ms = static_cast<T>(mm * s1 * ui);
    if (mm == 0) {  // one column: both signs of m write the same value
      c = s = kIS2;
      mc = ms = T(0);
    }
    const T xr = static_cast<T>(ux * ui), yr = static_cast<T>(uy * ui);
    OrdChain<T> chain{static_cast<T>(uz), static_cast<T>(ux * ux + uy * uy)};
    T g0 = T(0), g1 = T(0), g2 = T(0);
    // LDS positions of columns k0 + m and k0 - m at degree l, of Y and dY's
    // x, y and z rows
    const int kb = l0 * l0 + l0;
    T* yp = sy + hy + p * K + kb + mm;
    T* ym = yp - 2 * mm;
    T* xp0 = sd + hd + 3 * p * K + kb + mm;
    T* xm0 = xp0 - 2 * mm;
    T *yp0 = xp0 + K, *ym0 = xm0 + K, *zp0 = yp0 + K, *zm0 = ym0 + K;
    const T* wpp = sg + hg + p * K + kb + mm;
    const T* wmp = wpp - 2 * mm;
    const T ir = static_cast<T>(ui), uzi = static_cast<T>(uz * ui);
    // YZ, XY: which outputs this thread forms
    auto walk = [&](auto yz_c, auto xy_c) {
      constexpr bool YZ = decltype(yz_c)::value, XY = decltype(xy_c)::value;
      constexpr bool DER = SD || BWD;
      T fl = T(l0);
      // N: the coefficients of degree l; inv: 1 / (l + 1 + m)
      auto degree = [&](int l, T N, T inv) {
#pragma clang fp contract(off)
        if (lane_on && l >= mm) {
          T wp = T(0), wm = T(0);
          if constexpr (BWD) {
            wp = *wpp;
            wm = mm == 0 ? T(0) : *wmp;
          }
          const T q = N * chain.p;
          if constexpr (SY && YZ) {
            *yp = q * c;
            *ym = q * s;
          }
          if constexpr (YZ && DER) {
            T dz = (N * chain.x) * chain.pl;
            if constexpr (NORM) dz = ord_fma(dz, ir, -((fl * uzi) * q));
            const T zp1 = dz * c, zm1 = dz * s;
            if constexpr (SD) {
              *zp0 = zp1;
              *zm0 = zm1;
            }
            if constexpr (BWD) g2 = ord_fma(wp, zp1, ord_fma(wm, zm1, g2));
          }
          if constexpr (XY && DER) {
            T E = N * chain.e;
            if constexpr (NORM) E = ord_fma(-fl, q, E);
            const T dx = xr * E, dy = yr * E;
            const T qc = q * mc, qs = q * ms;
            const T xp1 = ord_fma(dx, c, qc), xm1 = ord_fma(dx, s, qs);
            const T yp1 = ord_fma(dy, c, -qs), ym1 = ord_fma(dy, s, qc);
            if constexpr (SD) {
              *xp0 = xp1;
              *xm0 = xm1;
              *yp0 = yp1;
              *ym0 = ym1;
            }
            if constexpr (BWD) {
              g0 = ord_fma(wp, xp1, ord_fma(wm, xm1, g0));
              g1 = ord_fma(wp, yp1, ord_fma(wm, ym1, g1));
            }
          }
          chain.template advance<XY && DER>(inv);
        }
        fl += T(1);
        const int step = 2 * l + 2;
        yp += step;
        ym += step;
        xp0 += step;
        xm0 += step;
        yp0 += step;
        ym0 += step;
        zp0 += step;
        zm0 += step;
        wpp += step;
        wmp += step;
      };
      // kOrdStep degrees per trip, the next trip's coefficients loaded before
      // this one's arithmetic
      T A[2 * kOrdStep], B[2 * kOrdStep];
#pragma unroll
      for (int u = 0; u < kOrdStep; ++u) {
        A[2 * u] = C.a[l0 + u][2 * mm];
        A[2 * u + 1] = C.a[l0 + u][2 * mm + 1];
      }
      for (int l = l0; l <= L; l += kOrdStep) {
#pragma unroll
        for (int u = 0; u < kOrdStep; ++u) {
          B[2 * u] = C.a[l + kOrdStep + u][2 * mm];
          B[2 * u + 1] = C.a[l + kOrdStep + u][2 * mm + 1];
        }
#pragma unroll
        for (int u = 0; u < kOrdStep; ++u)
          if (l + u <= L) degree(l + u, A[2 * u], u + 1 < kOrdStep ? A[(2 * u + 3) % (2 * kOrdStep)] : B[1]);
#pragma unroll
        for (int u = 0; u < 2 * kOrdStep; ++u) A[u] = B[u];
      }
    };
    if constexpr (SPLIT) {
      if (part == 0)
        walk(std::true_type{}, std::false_type{});
      else
        walk(std::false_type{}, std::true_type{});
    } else {
      walk(std::true_type{}, std::true_type{});
    }
    if constexpr (BWD) {
      if (lane_on) {
        if (!SPLIT || part == 1) {
          sacc[m * PT + p] = g0;
          sacc[(L + 1 + m) * PT + p] = g1;
        }
        if (!SPLIT || part == 0) sacc[(2 * (L + 1) + m) * PT + p] = g2;
      }
    }
    __syncthreads();
    if constexpr (BWD) {
      if (tid < 3 * np) {  // sums over the orders, in order
        const int a = tid % 3, pp = tid / 3;
        const T* sp = sacc + a * (L + 1) * PT + pp;
        T v = T(0);
        for (int j = 0; j <= L; ++j) v += sp[j * PT];
        // e3nn: the points are (z, x, y), so the second axis' sum is d/dx
        static_cast<T*>(P.gxyz)[(p0 + pp) * 3 + (P.conv == 0 ? a : (a + 2) % 3)] = v;
      }
    }
    if constexpr (SY) ord_copy_out(sy, hy, gy, np * K, tid, nt);
    if constexpr (SD) ord_copy_out(sd, hd, gd, 3 * np * K, tid, nt);
    if (tile + gridDim.x < tiles) __syncthreads();  // another tile: every read of this one is done
  }
}

}  // namespace sph
