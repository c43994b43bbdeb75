// Double backward for compile-time degrees (sph_dbord.inl holds the rest): for
// v = dL'/d(gxyz),
//   ggY[i,k]   = sum_a v[i,a] dY[i,a,k]
//   gxyz2[i,b] = sum_k gY[i,k] sum_a v[i,a] d2Y[i,k]/(dx_a dx_b)
// One lane per point, 64-point tiles.  Nothing of the Hessian reaches memory:
// for every order the lane forms the Hessian-vector products of its two
// columns in registers from three consecutive rows of the folded polynomials
// and accumulates gY_k H_k v; ggY takes gY's place in the tile.  The degrees
// are unrolled, with their coefficients as literals, and split between the
// tile's waves.
//
// Bound by memory: w (2 K + 9) bytes per point.  1e6 points, normalised,
// against run-time degrees with tables of eight terms per order: float l_max 4
// 51 -> 41 us, l_max 6 94 -> 73 (5.9 TB/s), l_max 8 182 -> 128, l_max 12 578 ->
// 347; double (500 000) l_max 4 62 -> 44, l_max 7 220 -> 97, l_max 8 280 -> 193
// (its registers spill; scaled harmonics 198 -> 143).
//
// Second derivatives by applying Eq. iter-deri twice:
//   H(Qt) v = ( Tm vx + x W, Tm vy + y W, W1 rho + W0 vz ),
//     rho = x vx + y vy,  W = W2 rho + W1 vz,
//     Tm = gxy Qt_{l-1}^{m+1}, W2 = h2 Qt_{l-2}^{m+2}, W1 = h1 Qt_{l-2}^{m+1},
//     W0 = h0 Qt_{l-2}^m;
//   grad c_m = m (c_{m-1}, -s_{m-1}, 0),  grad s_m = m (s_{m-1}, c_{m-1}, 0),
//   H(c_m) = m(m-1) [[c_{m-2}, -s_{m-2}], [-s_{m-2}, -c_{m-2}]] (x-y block),
//   H(s_m) = m(m-1) [[s_{m-2},  c_{m-2}], [ c_{m-2}, -s_{m-2}]],
// and the product rule H(Qt t) v = t H(Qt) v + grad Qt (grad t . v)
//   + grad t (grad Qt . v) + Qt H(t) v.
// Normalised harmonics Y(x) = Yt(x/r): with u = x/r, g = grad Yt(u),
//   grad Y = (g - l Yt u) / r,
//   H Y v = [ H Yt v - l (g (u.v) + u (g.v)) - l Yt v + l(l+2) Yt u (u.v) ] / r^2.
#pragma once

#include "sph_device.hpp"
#include "sph_launch.hpp"

namespace sph {

// Waves per tile: two from l_max 2 (float, 1e6 points, one / two / four: l_max
// 1 12.2 / - / - us, l_max 3 33 / 29 / 33, l_max 6 87 / 73 / 80, l_max 8 - / 128
// / 150), four from float l_max 10 (10 - / 214 / 205, 12 - / 355 / 347) and for
// double scaled harmonics at l_max 8 (143, over 171 with two).
template <typename T>
constexpr int dbwd_waves(int L, bool normalize) {
  if (sizeof(T) == 8) return L < 2 ? 1 : (L >= 8 && !normalize ? 4 : 2);
  return L < 2 ? 1 : (L >= 10 ? 4 : 2);
}
template <typename T>
constexpr size_t dbwd_lds_bytes(int L, int waves) {
  return sizeof(T) * static_cast<size_t>(kWave) * static_cast<size_t>(row_stride<T>((L + 1) * (L + 1), true) + 3 * (waves - 1));
}

template <typename T>
struct DbwdAcc {
  T hx, hy, hz;  // sum_k gY_k H_k v (at the evaluation point)
};

// Degrees [LA, LB) of one point: row[k] = gY[k], replaced by ggY[k] where
// write_gg.
template <typename T, bool NORM, int LA, int LB>
__device__ __forceinline__ void dbwd_degrees(const Point<T>& pt, T vx, T vy, T vz, T* st, int o, bool write_gg,
                                             DbwdAcc<T>& A) {
  if constexpr (LA < LB) {
    constexpr int MM = LB - 1;
    const CoefTable<T>& C = coef<T>();
    constexpr T kIS2 = T(kInvSqrt2d);
    const T ex = pt.ex, ey = pt.ey;
    T ez = pt.ez;
    const T rho = ex * vx + ey * vy;
    const T uv = rho + ez * vz;  // u.v (normalised: ex = u)
    // c_m, s_m and tv = grad(c_m).v, grad(s_m).v; H(c_m) v = (hA, -hB) and
    // H(s_m) v = (hB, hA) with hA = m tvc_{m-1}, hB = m tvs_{m-1}
    T c[MM + 1], s[MM + 1], tvc[MM + 1], tvs[MM + 1];
    c[0] = T(1);
    s[0] = T(0);
    tvc[0] = tvs[0] = T(0);
#pragma unroll
    for (int m = 1; m <= MM; ++m) {
      s[m] = ex * s[m - 1] + ey * c[m - 1];
      c[m] = ex * c[m - 1] - ey * s[m - 1];
      tvc[m] = T(m) * (c[m - 1] * vx - s[m - 1] * vy);
      tvs[m] = T(m) * (s[m - 1] * vx + c[m - 1] * vy);
    }
    T pp[MM + 3], prev[MM + 3], cur[MM + 3];
    if constexpr (LA >= 2) q_row<T, MM>(LA - 2, ez, pt.rxy2, pp);
    if constexpr (LA >= 1) q_row<T, MM>(LA - 1, ez, pt.rxy2, prev);
    T hx0 = A.hx, hy0 = A.hy, hz0 = A.hz;
#pragma unroll
    for (int l = LA; l < LB; ++l) {
      q_row<T, MM>(l, ez, pt.rxy2, cur);
      T* row = st + o;
      const int k0 = l * l + l;
      T Sgv = T(0), Sgx = T(0), Sgy = T(0), Sgz = T(0), Sy = T(0);
      const T luv = T(l) * uv;  // normalised: grad Y . v = (grad Yt . v - l (u.v) Yt) / r
#pragma unroll
      for (int m = 0; m <= MM; ++m) {
        if (m > l) continue;  // no early exit: keeps the loop fully unrolled
        const T q = cur[m];
        T Tm = T(0), Cz = T(0), W2 = T(0), W1 = T(0), W0 = T(0);
        if (m <= l - 2) Tm = C.gxy[l][m] * prev[m + 1];
        if (m <= l - 1) Cz = C.gz[l][m] * prev[m];
        if (m <= l - 4) W2 = C.h2[l][m] * pp[m + 2];
        if (m <= l - 3) W1 = C.h1[l][m] * pp[m + 1];
        if (m <= l - 2) W0 = C.h0[l][m] * pp[m];
        const T Qx = ex * Tm, Qy = ey * Tm;  // grad Qt = (Qx, Qy, Cz)
        const T W = W2 * rho + W1 * vz;
        const T Hx = Tm * vx + ex * W;  // H(Qt) v
        const T Hy = Tm * vy + ey * W;
        const T Hz = W1 * rho + W0 * vz;
        const T gQv = Tm * rho + Cz * vz;  // grad Qt . v
        // Everything accumulated is linear in the weights, so the columns k0 + m
        // (t = c_m, grad t = (mc, -ms), H(t) v = (hA, -hB)) and k0 - m (t = s_m,
        // grad t = (ms, mc), H(t) v = (hB, hA)) of one order fold into P = wp c +
        // wm s and five like combinations before they meet the row's terms.
        if (m == 0) {
          const T P = row[k0] * kIS2;
          if (write_gg) {
            T gg = gQv;
            if constexpr (NORM) gg = (gg - luv * q) * pt.inv_r;
            row[k0] = gg * kIS2;
          }
          hx0 += Hx * P;
          hy0 += Hy * P;
          hz0 += Hz * P;
          if constexpr (NORM) {
            Sgx += Qx * P;
            Sgy += Qy * P;
            Sgz += Cz * P;
            Sgv += gQv * P;
            Sy += q * P;
          }
        } else {
          const int kp = k0 + m, km = k0 - m;
          const T wp = row[kp], wm = row[km];
          const T mc = T(m) * c[m - 1], ms = T(m) * s[m - 1];
          const T hA = T(m) * tvc[m - 1], hB = T(m) * tvs[m - 1];
          if (write_gg) {  // grad Y . v of each column
            T ggp = c[m] * gQv + q * tvc[m], ggm = s[m] * gQv + q * tvs[m];
            if constexpr (NORM) {
              ggp = (ggp - luv * (q * c[m])) * pt.inv_r;
              ggm = (ggm - luv * (q * s[m])) * pt.inv_r;
            }
            row[kp] = ggp;
            row[km] = ggm;
          }
          const T P = wp * c[m] + wm * s[m];
          const T Pt = wp * tvc[m] + wm * tvs[m];
          const T Pm = wp * mc + wm * ms;
          const T Pn = wm * mc - wp * ms;
          const T Ph = wp * hA + wm * hB;
          const T Pk = wm * hA - wp * hB;
          hx0 += Hx * P + Qx * Pt + gQv * Pm + q * Ph;
          hy0 += Hy * P + Qy * Pt + gQv * Pn + q * Pk;
          hz0 += Hz * P + Cz * Pt;
          if constexpr (NORM) {
            Sgx += Qx * P + q * Pm;
            Sgy += Qy * P + q * Pn;
            Sgz += Cz * P;
            Sgv += gQv * P + q * Pt;
            Sy += q * P;
          }
        }
      }
      if constexpr (NORM) {
        const T fl = T(l);
        const T a = fl * (fl + T(2)) * Sy * uv;
        hx0 += -fl * (Sgx * uv + ex * Sgv) - fl * Sy * vx + a * ex;
        hy0 += -fl * (Sgy * uv + ey * Sgv) - fl * Sy * vy + a * ey;
        hz0 += -fl * (Sgz * uv + ez * Sgv) - fl * Sy * vz + a * ez;
      }
      copy_row<T, MM>(l, prev, pp);
      copy_row<T, MM>(l, cur, prev);
      // The next degree starts after this one (see vjp_degrees): interleaved,
      // the unrolled degrees hold most of the row in registers.
      asm volatile("" : "+v"(ez), "+v"(o), "+v"(hx0), "+v"(hy0), "+v"(hz0));
    }
    A.hx = hx0;
    A.hy = hy0;
    A.hz = hz0;
  }
}

template <typename T, int LT, bool NORM, int DS, int... Hs>
__device__ __forceinline__ void dbwd_parts(std::integer_sequence<int, Hs...>, int h, const Point<T>& pt, T vx, T vy,
                                           T vz, T* st, int o, bool write_gg, DbwdAcc<T>& A) {
  ((h == Hs ? dbwd_degrees<T, NORM, degree_split(LT, DS, Hs), degree_split(LT, DS, Hs + 1)>(pt, vx, vy, vz, st, o,
                                                                                           write_gg, A)
            : void()),
   ...);
}

// l_max = LT at compile time, 64-point tiles.  The degrees of a tile are split
// between the block's DS waves (the branch is uniform per wave), which copy
// the tile together; waves past the first hand their Hessian sums over through
// LDS.  Dynamic LDS: dbwd_lds_bytes.
template <typename T, int LT, bool NORM, int DS>
__global__ __launch_bounds__(kWave * DS) void k_dbwd(DbwdParams P) {
  constexpr int NT = kWave * DS;
  constexpr int K = (LT + 1) * (LT + 1);
  constexpr int S = row_stride<T>(K, true);
  extern __shared__ __align__(16) unsigned char smem[];
  T* st = reinterpret_cast<T*>(smem);
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int h = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int64_t p0 = static_cast<int64_t>(blockIdx.x) * kWave;
  if (p0 >= P.n) return;
  const int np = static_cast<int>(P.n - p0 < kWave ? P.n - p0 : kWave);
  const T* src = static_cast<const T*>(P.gY) + p0 * K;
  copy_in<NT>(st, S, src, K, K, np, tid, aligned16(src));
  T x = T(0), y = T(0), z = T(0), vx = T(0), vy = T(0), vz = T(0);
  if (lane < np) {
    const T* q = static_cast<const T*>(P.xyz) + (p0 + lane) * 3;
    x = q[0];
    y = q[1];
    z = q[2];
    const T* w = static_cast<const T*>(P.v) + (p0 + lane) * 3;
    vx = w[0];
    vy = w[1];
    vz = w[2];
  }
  const Point<T> pt = make_point<T, NORM>(x, y, z);
  const bool write_gg = P.ggY != nullptr;
  DbwdAcc<T> A{T(0), T(0), T(0)};
  __syncthreads();
  dbwd_parts<T, LT, NORM, DS>(std::make_integer_sequence<int, DS>{}, h, pt, vx, vy, vz, st, lane * S, write_gg, A);
  T* sacc = st + kWave * S;
  if constexpr (DS > 1) {
    if (h > 0) {
      sacc[(3 * h - 3) * kWave + lane] = A.hx;
      sacc[(3 * h - 2) * kWave + lane] = A.hy;
      sacc[(3 * h - 1) * kWave + lane] = A.hz;
    }
  }
  __syncthreads();
  if (write_gg) {
    T* dst = static_cast<T*>(P.ggY) + p0 * K;
    copy_out<NT>(st, S, dst, K, K, np, tid, aligned16(dst));
  }
  if (h > 0) return;
#pragma unroll
  for (int i = 0; i < DS - 1; ++i) {
    A.hx += sacc[3 * i * kWave + lane];
    A.hy += sacc[(3 * i + 1) * kWave + lane];
    A.hz += sacc[(3 * i + 2) * kWave + lane];
  }
  if (P.gxyz2 != nullptr && lane < np) {
    T s = T(1);
    if constexpr (NORM) s = pt.inv_r * pt.inv_r;
    T* g = static_cast<T*>(P.gxyz2) + (p0 + lane) * 3;
    g[0] = A.hx * s;
    g[1] = A.hy * s;
    g[2] = A.hz * s;
  }
}

}  // namespace sph
