// Double backward for degrees past the compile-time kernels (see sph_dbwd.inl
// for the outputs): one lane per (point, order), see sph_ord.inl.
//
// A lane walks the degrees upward at fixed order with the recursion carried to
// second derivatives (HessChain), and its sums over the degrees are of
// gY times the few quantities that depend on the degree (q, T, Z, W, V, U and
// four more weighted by l); the order's factors, v and u enter once, after the
// last degree.  ggY takes gY's place in the LDS tile.  Where a sum is not
// finite the lane forms its columns' H v one by one instead, so that an
// infinite gY gives its products with them; and where the scaled harmonics may
// be past the type's range (see HessChain) its columns of ggY as well.
//
// Against one lane per point with groups of degrees staged through LDS: float
// l_max 16, 100 000 points 442 -> 88 us, l_max 32 1769 -> 267 (3.3 TB/s);
// double l_max 9, 500 000 points 614 -> 339, l_max 12 1020 -> 477, l_max 32,
// 50 000 points 1387 -> 244.  Below, the lanes' own set-up and the waves of
// few orders cost more than they give (float l_max 8 284 us, 128 in k_dbwd).
#pragma once

#include "sph_ord.inl"

namespace sph {

// Tile row stride: odd, so that the lanes of one order hit distinct banks.
__host__ __device__ constexpr int dbord_stride(int L) { return (L + 1) * (L + 1) | 1; }

template <typename T>
__host__ __device__ constexpr size_t dbord_lds_bytes(int L, int points) {
  return sizeof(T) * (static_cast<size_t>(ord_block<T>(points * dbord_stride(L))) + (3u * (L + 1) + 1u) * points);
}

// cnt elements of rows of K between global g and LDS rows of K + 1 (K a whole
// number of vectors): as vectors where g is aligned.
template <typename T, bool IN>
__device__ __forceinline__ void dbord_copy_padded(T* st, T* g, int cnt, int K, bool vec, int tid, int nt) {
  using V = typename Vec16<T>::type;
  constexpr int W = Vec16<T>::n;
  constexpr int NB = 4;
  if (vec) {
    V* gv = reinterpret_cast<V*>(g);
    const int KV = K / W, nv = cnt / W;
    for (int i0 = tid; i0 < nv; i0 += nt * NB) {
      V v[NB];
      if constexpr (IN) {
#pragma unroll
        for (int u = 0; u < NB; ++u)
          if (i0 + u * nt < nv) v[u] = __builtin_nontemporal_load(gv + i0 + u * nt);
      }
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int i = i0 + u * nt;
        if (i < nv) {
          T* s = st + i * W + i / KV;
#pragma unroll
          for (int t = 0; t < W; ++t) {
            if constexpr (IN)
              s[t] = v[u][t];
            else
              v[u][t] = s[t];
          }
        }
      }
      if constexpr (!IN) {
#pragma unroll
        for (int u = 0; u < NB; ++u)
          if (i0 + u * nt < nv) __builtin_nontemporal_store(v[u], gv + i0 + u * nt);
      }
    }
  } else {
    for (int i = tid; i < cnt; i += nt) {
      if constexpr (IN)
        st[i + i / K] = g[i];
      else
        g[i] = st[i + i / K];
    }
  }
}

// Points per tile: the most that fill their waves best, up to four waves and
// 80 KiB of LDS (double l_max 32 7 points 244 us, 6 271, 3 280; l_max 24 10
// points 153, 8 174; float l_max 16 15 points 88, 12 105).
template <typename T>
constexpr int dbord_points(int L) {
  int best = 1, fill = 0;
  for (int p = 1; p * (L + 1) <= 256 && dbord_lds_bytes<T>(L, p) <= 80 * 1024; ++p) {
    const int used = p * (L + 1), f = 1000 * used / ((used + 63) / 64 * 64);
    if (f >= fill) {
      best = p;
      fill = f;
    }
  }
  return best;
}

// P.tile points per block, P.tile (l_max + 1) lanes rounded up to whole waves.
// Dynamic LDS: dbord_lds_bytes.  A grid-stride loop over tiles, so any grid is
// correct.
template <typename T, bool NORM>
__global__ __launch_bounds__(256) void k_dbord(DbwdParams P) {
  constexpr T kIS2 = T(kInvSqrt2d);
  extern __shared__ __align__(16) unsigned char smem[];
  const int L = P.L;
  const int K = (L + 1) * (L + 1), S = dbord_stride(L);
  const bool padded = S != K;
  const int PT = P.tile;
  T* st = reinterpret_cast<T*>(smem);
  T* sacc = st + ord_block<T>(PT * S);
  T* sir = sacc + 3 * (L + 1) * PT;  // 1/r of each point
  const int tid = threadIdx.x, nt = blockDim.x;
  const OrdTable<T>& C = ord_table<T>(0);
  const int m = tid / PT, p = tid - m * PT;
  const bool lane_on = m <= L;
  const int mm = lane_on ? m : L;
  const int lw = __builtin_amdgcn_readfirstlane(tid / kWave * kWave / PT);
  const int l0 = lw <= L ? lw : L + 1;
  const int64_t tiles = (P.n + PT - 1) / PT;
  for (int64_t tile = xcd_slot(blockIdx.x, gridDim.x); tile < tiles; tile += gridDim.x) {
    const int64_t p0 = tile * PT;
    const int np = static_cast<int>(P.n - p0 < PT ? P.n - p0 : PT);
    const int pp = p < np ? p : np - 1;
    const T* xp = static_cast<const T*>(P.xyz) + (p0 + pp) * 3;
    const T* vp = static_cast<const T*>(P.v) + (p0 + pp) * 3;
    const T xin = xp[0], yin = xp[1], zin = xp[2];
    const T v0 = vp[0], v1 = vp[1], v2 = vp[2];
    const T* gg = static_cast<const T*>(P.gY) + p0 * K;
    T* go = P.ggY != nullptr ? static_cast<T*>(P.ggY) + p0 * K : nullptr;
    const int hg = padded ? 0 : ord_shift(gg);
    if (padded)
      dbord_copy_padded<T, true>(st, const_cast<T*>(gg), np * K, K, ord_shift(gg) == 0, tid, nt);
    else
      ord_copy_in(st, hg, gg, np * K, tid, nt);
    const Point<T> pt = make_point<T, NORM>(xin, yin, zin);
    // the evaluation point and its powers in double, as in k_ord
    double ux = xin, uy = yin, uz = zin, ui = 1.0;
    if constexpr (NORM) {
      ui = static_cast<double>(pt.inv_r);
      if constexpr (!std::is_same_v<T, double>) {
        const double rr = ux * ux + uy * uy + uz * uz;
        ui = pt.inv_r == T(0) ? 0.0 : ui * (1.5 - 0.5 * rr * ui * ui);
      }
      ux *= ui;
      uy *= ui;
      uz *= ui;
    }
    double c2 = 1.0, s2 = 0.0;
    {
      const int ex = mm >= 2 ? mm - 2 : 0;
      double bc = ux, bs = uy;
#pragma unroll
      for (int b = 0; b < 5; ++b) {
        if ((ex >> b) & 1) {
          const double t = c2 * bc - s2 * bs;
          s2 = c2 * bs + s2 * bc;
          c2 = t;
        }
        const double t = bc * bc - bs * bs;
        bs = 2.0 * bc * bs;
        bc = t;
      }
    }
    double c1 = 1.0, s1 = 0.0;
    if (mm >= 2) {
      c1 = c2 * ux - s2 * uy;
      s1 = c2 * uy + s2 * ux;
    }
    const double c0 = c1 * ux - s1 * uy, s0 = c1 * uy + s1 * ux;
    const double fm = mm, fmm = mm * (mm - 1);
    T tp = static_cast<T>(c0), tpx = static_cast<T>(fm * c1), tpy = static_cast<T>(-fm * s1);
    T tm = static_cast<T>(s0), tmx = -tpy, tmy = tpx;
    const T A = static_cast<T>(fmm * c2), B = static_cast<T>(fmm * s2);
    if (mm == 0) {
      tp = tm = kIS2;
      tpx = tpy = tmx = tmy = T(0);
    }
    const T x = static_cast<T>(ux), y = static_cast<T>(uy), z = static_cast<T>(uz);
    const T ir = static_cast<T>(ui);
    const T rho2 = static_cast<T>(ux * ux + uy * uy);
    const T vx = v0 * ir, vy = v1 * ir, vz = v2 * ir;
    const T rho = x * vx + y * vy, uv = rho + z * vz;
    T tvp = tpx * vx + tpy * vy, tvm = tmx * vx + tmy * vy;
    // H(c_m) v and H(s_m) v
    T hpx = A * vx - B * vy, hpy = -(B * vx + A * vy);
    T hmx = B * vx + A * vy, hmy = A * vx - B * vy;
    if (mm == 0) tvp = tvm = hpx = hpy = hmx = hmy = T(0);  // (also of an infinite v)
    const bool far = !NORM && !(rho2 + z * z <= static_cast<T>(P.reach2));
    __syncthreads();
    const int kb = l0 * l0 + l0;
    T* basp = st + hg + p * S + kb + mm;
    T* basm = basp - 2 * mm;
    T fl = T(l0);
    HessChain<T> ch{z, rho2};
    // sums over the degrees, per sign: of gY times q, T, Z, W, V, U and, for
    // the normalised harmonics, l q, l(l+2) q, l T, l Z
    T Sq[2] = {}, Sl[2] = {}, Sll[2] = {}, St[2] = {}, Slt[2] = {}, Sz[2] = {}, Slz[2] = {}, Sw[2] = {}, Sv[2] = {},
      Su[2] = {};
    auto degree = [&](int l, T N, T inv) {
      if (lane_on && l >= mm) {
        const T gp = *basp, gm = mm == 0 ? T(0) : *basm;
        const T q = N * ch.p, Tm = N * ch.e, Wn = N * ch.w;
        const T Nx = N * ch.x;
        const T Z = Nx * ch.p1, V = Nx * ch.e1, U = Nx * ((ch.x - T(1)) * ch.p2);
        T G = Tm * rho + Z * vz;
        if constexpr (NORM) G -= (fl * uv) * q;
        *basp = tp * G + q * tvp;
        *basm = tm * G + q * tvm;
        auto sum = [&](int i, T a) {
          Sq[i] += a * q;
          St[i] += a * Tm;
          Sz[i] += a * Z;
          Sw[i] += a * Wn;
          Sv[i] += a * V;
          Su[i] += a * U;
          if constexpr (NORM) {
            const T al = a * fl;
            Sl[i] += al * q;
            Sll[i] += (al * (fl + T(2))) * q;
            Slt[i] += al * Tm;
            Slz[i] += al * Z;
          }
        };
        sum(0, gp);
        sum(1, gm);
        ch.advance(inv, MulPlain{});
      }
      fl += T(1);
      basp += 2 * l + 2;
      basm += 2 * l + 2;
    };
    T Ac[2 * kOrdStep], Bc[2 * kOrdStep];
#pragma unroll
    for (int u = 0; u < kOrdStep; ++u) {
      Ac[2 * u] = C.a[l0 + u][2 * mm];
      Ac[2 * u + 1] = C.a[l0 + u][2 * mm + 1];
    }
#pragma unroll 1
    for (int l = l0; l <= L; l += kOrdStep) {
#pragma unroll
      for (int u = 0; u < kOrdStep; ++u) {
        Bc[2 * u] = C.a[l + kOrdStep + u][2 * mm];
        Bc[2 * u + 1] = C.a[l + kOrdStep + u][2 * mm + 1];
      }
#pragma unroll
      for (int u = 0; u < kOrdStep; ++u)
        if (l + u <= L) degree(l + u, Ac[2 * u], u + 1 < kOrdStep ? Ac[(2 * u + 3) % (2 * kOrdStep)] : Bc[1]);
#pragma unroll
      for (int u = 0; u < 2 * kOrdStep; ++u) Ac[u] = Bc[u];
    }
    // one sign's H v from its sums
    T hx = T(0), hy = T(0), hz = T(0);
    auto apply = [&](int i, T t, T tx, T ty, T tv, T Hx, T Hy) {
      const T gv = St[i] * rho + Sz[i] * vz;  // grad Qt . v
      const T ww = Sw[i] * rho + Sv[i] * vz;
      const T xt = St[i] * tv;
      hx += t * (St[i] * vx + x * ww) + x * xt + tx * gv + Sq[i] * Hx;
      hy += t * (St[i] * vy + y * ww) + y * xt + ty * gv + Sq[i] * Hy;
      hz += t * (Sv[i] * rho + Su[i] * vz) + Sz[i] * tv;
      if constexpr (NORM) {
        // - l (u.v) g - l (g.v) u - l Yt v + l(l+2) Yt (u.v) u
        const T lgx = x * Slt[i] * t + Sl[i] * tx, lgy = y * Slt[i] * t + Sl[i] * ty, lgz = Slz[i] * t;
        const T b = (Slt[i] * rho + Slz[i] * vz) * t + Sl[i] * tv - Sll[i] * t * uv;
        const T ly = Sl[i] * t;
        hx -= uv * lgx + b * x + ly * vx;
        hy -= uv * lgy + b * y + ly * vy;
        hz -= uv * lgz + b * z + ly * vz;
      }
    };
    apply(0, tp, tpx, tpy, tvp, hpx, hpy);
    apply(1, tm, tmx, tmy, tvm, hmx, hmy);
    if (lane_on && (P.gxyz2 != nullptr || far)) {
      // not finite (an infinite or very large gY): column by column, so that
      // each column's product with its H v decides, not a sum's with a factor
      if (far || !(hx - hx == T(0) && hy - hy == T(0) && hz - hz == T(0))) {
        hx = hy = hz = T(0);
        const T* gp = gg + static_cast<int64_t>(pp) * K;
        T* gt = st + hg + p * S;
        const std::conditional_t<NORM, MulPlain, MulZero> mul;
        ch = HessChain<T>{z, rho2};
        fl = T(mm);
#pragma unroll 1
        for (int l = mm; l <= L; ++l) {
          const T N = C.a[l][2 * mm];
          const T q = N * ch.p, Tm = N * ch.e, Wn = N * ch.w, Nx = N * ch.x;
          const T Z = Nx * ch.p1, V = Nx * ch.e1, U = Nx * ((ch.x - T(1)) * ch.p2);
          const T gQv = mul(Tm, rho) + mul(Z, vz), ww = mul(Wn, rho) + mul(V, vz);
          auto col = [&](int k, T t, T tx, T ty, T tv, T Hx, T Hy) {
            T ax = mul(t, mul(Tm, vx) + mul(x, ww)) + mul(mul(x, Tm), tv) + mul(tx, gQv) + mul(q, Hx);
            T ay = mul(t, mul(Tm, vy) + mul(y, ww)) + mul(mul(y, Tm), tv) + mul(ty, gQv) + mul(q, Hy);
            T az = mul(t, mul(V, rho) + mul(U, vz)) + mul(Z, tv);
            if constexpr (NORM) {
              const T Yt = q * t, gx = x * Tm * t + q * tx, gy = y * Tm * t + q * ty, gz = Z * t;
              const T b = fl * (gQv * t + q * tv) - fl * (fl + T(2)) * uv * Yt;
              ax -= fl * (uv * gx + Yt * vx) + b * x;
              ay -= fl * (uv * gy + Yt * vy) + b * y;
              az -= fl * (uv * gz + Yt * vz) + b * z;
            }
            const T a = gp[k];
            hx += a * ax;
            hy += a * ay;
            hz += a * az;
            if (far) gt[k] = mul(t, gQv) + mul(q, tv);
          };
          const int k0 = l * l + l;
          col(k0 + mm, tp, tpx, tpy, tvp, hpx, hpy);
          if (mm > 0) col(k0 - mm, tm, tmx, tmy, tvm, hmx, hmy);
          ch.advance(C.a[l + 1][2 * mm + 1], mul);
          fl += T(1);
        }
      }
      if (m == 0) sir[p] = ir;
      sacc[m * PT + p] = hx;
      sacc[(L + 1 + m) * PT + p] = hy;
      sacc[(2 * (L + 1) + m) * PT + p] = hz;
    }
    __syncthreads();
    if (P.gxyz2 != nullptr) {
      for (int i = tid; i < 3 * np; i += nt) {  // sums over the orders, in order
        const int a = i % 3, q = i / 3;
        const T* sp = sacc + a * (L + 1) * PT + q;
        T s = T(0);
        for (int j = 0; j <= L; ++j) s += sp[j * PT];
        // the second 1/r last: a sum that it takes past the type's range is an
        // infinity, not the difference of the orders' infinities
        static_cast<T*>(P.gxyz2)[(p0 + q) * 3 + a] = s * sir[q];
      }
    }
    if (P.ggY != nullptr) {
      if (padded) {
        dbord_copy_padded<T, false>(st, go, np * K, K, ord_shift(go) == 0, tid, nt);
      } else if (ord_shift(go) == hg) {
        ord_copy_out(st, hg, go, np * K, tid, nt);
      } else {  // another alignment than gY's
        for (int i = tid; i < np * K; i += nt) go[i] = st[hg + i];
      }
    }
    if (tile + gridDim.x < tiles) __syncthreads();
  }
}

}  // namespace sph
