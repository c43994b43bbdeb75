// Backward from the points (vector-Jacobian product without stored
// derivatives): for gY = dL/dY,
//   gxyz[i,a] = sum_k gY[i,k] dY_k/dx_a(xyz[i])
// with the derivatives formed in registers.
//
// Bound by the read of gY: it moves w (K + 6) bytes per point where the
// contraction of stored derivatives moves w (4 K + 3) and its forward 3 K w
// more.  Float, normalised: l_max 8, 1e6 points 54 us (6.4 TB/s) against 200
// us for k_bwd; l_max 6, 4e6 points 133 us (6.6 TB/s) against 541; double
// l_max 8, 300 000 points 41 us against 128.
//
// One lane per point, 64-point tiles.  The tile's gY rows arrive in LDS by
// coalesced 16-byte loads (all of a thread's loads in flight at once; they
// overlap the order-m tables), then every lane walks its own row: a
// degree's row of Qt (Eq. iter-q-alt) and the previous one give the
// derivatives of every column (Eq. iter-deri and the product rule), each
// multiplied by its gY as soon as it is formed.  The degrees of a tile are
// split between the block's DS waves, which add their sums in LDS.
#pragma once

#include "sph_device.hpp"
#include "sph_fwd.inl"
#include "sph_launch.hpp"

namespace sph {

constexpr int kVjpPoints = kWave;  // points per tile

// Waves per tile.  One for l_max <= 3 (l_max 3, float, 1e6 points: 13.4 us
// against 14.6 with two), four for double l_max 8, where two waves spill at
// two per SIMD (300 000 points: 41 us against 46 at one per SIMD), else two
// (float l_max 12, 500 000 points: 68 us against 140 with one; l_max 6, 4e6
// points: 133, 149 with four).
template <typename T>
constexpr int vjp_waves(int LT) {
  return LT <= 3 ? 1 : (!std::is_same_v<T, float> && LT >= 8 ? 4 : 2);
}

// LDS row stride (elements): odd, so the lanes' reads of one column of their
// rows hit distinct banks.
constexpr int vjp_stride(int K) { return K | 1; }

// Adds the degrees [LA, LB) of one point to g: st[o + k] = gY[k].
//   scaled derivatives, with Tm = gxy Qt_{l-1}^{m+1}, Cm = gz Qt_{l-1}^m and
//   D = Tm - l Qt_l^m (normalised; the chain rule's -l u_a Y folded in),
//   D = Tm (scaled):
//     d/dx = x D {c_m, s_m} + m Qt_l^m {c_{m-1}, s_{m-1}}
//     d/dy = y D {c_m, s_m} + m Qt_l^m {-s_{m-1}, c_{m-1}}
//     d/dz = (Cm - l z Qt_l^m) {c_m, s_m}
// (normalised: the caller multiplies the sums by 1/r).
template <typename T, bool NORM, bool E3, int LA, int LB>
__device__ __forceinline__ void vjp_degrees(const Point<T>& pt, const T* st, int o, int conv, T (&g)[3]) {
  constexpr int MM = LB - 1;
  const CoefTable<T>& C = coef<T>();
  constexpr T kIS2 = T(kInvSqrt2d);
  const T ex = pt.ex, ey = pt.ey;
  T ez = pt.ez;
  T c[MM + 1], s[MM + 1], mc[MM + 1], ms[MM + 1];
  c[0] = T(1);
  s[0] = T(0);
  mc[0] = ms[0] = T(0);
#pragma unroll
  for (int m = 1; m <= MM; ++m) {
    s[m] = ex * s[m - 1] + ey * c[m - 1];
    c[m] = ex * c[m - 1] - ey * s[m - 1];
    mc[m] = T(m) * c[m - 1];
    ms[m] = T(m) * s[m - 1];
  }
  T prev[MM + 3], cur[MM + 3];
  if constexpr (LA >= 1) q_row<T, MM>(LA - 1, ez, pt.rxy2, prev);
  T xs = T(0), ys = T(0), zs = T(0);  // E3: the degrees done, scaled
  T x0 = T(0), y0 = T(0), z0 = T(0), x1 = T(0), y1 = T(0), z1 = T(0);
#pragma unroll
  for (int l = LA; l < LB; ++l) {
    q_row<T, MM>(l, ez, pt.rxy2, cur);
    const int k0 = l * l + l;
    const T lz = T(l) * ez;
#pragma unroll
    for (int m = 0; m <= MM; ++m) {
      if (m > l) continue;  // no early exit: keeps the loop fully unrolled
      const T q = cur[m];
      T D = T(0), e = T(0);
      if (m <= l - 2) D = C.gxy[l][m] * prev[m + 1];
      if (m <= l - 1) e = C.gz[l][m] * prev[m];
      if constexpr (NORM) {
        D -= T(l) * q;
        e -= lz * q;
      }
      const T dx = ex * D, dy = ey * D;
      if (m == 0) {
        const T w = st[o + k0] * kIS2;
        x0 += w * dx;
        y0 += w * dy;
        z0 += w * e;
      } else {
        const T wp = st[o + k0 + m], wm = st[o + k0 - m];
        const T qc = q * mc[m], qs = q * ms[m];
        x0 += wp * (dx * c[m] + qc);
        y0 += wp * (dy * c[m] - qs);
        z0 += wp * (e * c[m]);
        x1 += wm * (dx * s[m] + qs);
        y1 += wm * (dy * s[m] + qc);
        z1 += wm * (e * s[m]);
      }
    }
    copy_row<T, MM>(l, cur, prev);
    if constexpr (E3) {
      const T cl = conv_scale<T>(conv, l);
      xs += cl * (x0 + x1);
      ys += cl * (y0 + y1);
      zs += cl * (z0 + z1);
      x0 = y0 = z0 = x1 = y1 = z1 = T(0);
    }
    // The next degree starts after this one: without this fence the unrolled
    // degrees interleave, hold most of the row in registers and spill (float
    // l_max 12, 500 000 points: 201 us against 68).
    if constexpr (E3)
      asm volatile("" : "+v"(ez), "+v"(o), "+v"(xs), "+v"(ys), "+v"(zs));
    else
      asm volatile("" : "+v"(ez), "+v"(o), "+v"(x0), "+v"(y0), "+v"(z0), "+v"(x1), "+v"(y1), "+v"(z1));
  }
  g[0] += E3 ? xs : x0 + x1;
  g[1] += E3 ? ys : y0 + y1;
  g[2] += E3 ? zs : z0 + z1;
}

// Wave h of the block: its part of the degrees (the branch is uniform per
// wave).
template <typename T, int LT, bool NORM, bool E3, int DS, int... Hs>
__device__ __forceinline__ void vjp_parts(std::integer_sequence<int, Hs...>, int h, const Point<T>& pt,
                                          const T* st, int o, int conv, T (&g)[3]) {
  ((h == Hs ? vjp_degrees<T, NORM, E3, degree_split(LT, DS, Hs), degree_split(LT, DS, Hs + 1)>(pt, st, o, conv, g) : void()), ...);
}

// l_max = LT at compile time.  E3: e3nn's convention (P.conv > 0), the sums
// scaled degree by degree; carried by every kernel that cost 1-10 % (float,
// 1e6 points: l_max 8 60 us against 56, l_max 3 16.1 against 14.5).  Dynamic LDS: 64 rows of vjp_stride(K)
// elements, then 3 * 64 sums per wave past the first.  gY may have any
// alignment: full tiles of 16-byte aligned arrays take the vector loads,
// others the general copy.
template <typename T, int LT, bool NORM, bool E3, int DS>
__global__ __launch_bounds__(kWave * DS) __attribute__((amdgpu_waves_per_eu(2))) void k_vjp(FwdParams P) {
  constexpr int K = (LT + 1) * (LT + 1);
  constexpr int S = vjp_stride(K);
  constexpr int W = Vec16<T>::n;
  constexpr int NT = kWave * DS;
  constexpr int NV = kWave * K / W;  // 16-byte vectors of a full tile
  constexpr int NB = (NV + NT - 1) / NT;
  static_assert((kWave * K) % W == 0, "a tile of whole vectors");
  using V = typename Vec16<T>::type;
  extern __shared__ __align__(16) unsigned char smem[];
  T* st = reinterpret_cast<T*>(smem);
  T* sacc = st + kWave * S;
  const int tid = threadIdx.x;
  const int lane = tid % kWave, h = tid / kWave;
  const T* xyz = static_cast<const T*>(P.xyz);
  const T* gY = static_cast<const T*>(P.gY);
  const bool aligned = aligned16(gY);
  for (int64_t tile = blockIdx.x; tile * kWave < P.n; tile += gridDim.x) {
    const int64_t p0 = tile * kWave;
    const int np = static_cast<int>(P.n - p0 < kWave ? P.n - p0 : kWave);
    const T* src = gY + p0 * K;
    const bool fast = aligned && np == kWave;
    V v[NB];
    if (fast) {
      const V* sv = reinterpret_cast<const V*>(src);
#pragma unroll
      for (int u = 0; u < NB; ++u)
        if (u < NV / NT || tid + u * NT < NV) v[u] = __builtin_nontemporal_load(sv + tid + u * NT);
    }
    const T* q = xyz + (p0 + (lane < np ? lane : np - 1)) * 3;
    const Point<T> pt = make_point<T, NORM>(q[0], q[1], q[2]);
    if (fast) {
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int i = tid + u * NT;
        if (u < NV / NT || i < NV) {
          if constexpr (S == K) {
            reinterpret_cast<V*>(st)[i] = v[u];
          } else {  // even K: a vector never crosses a row
            T* d = st + (i / (K / W)) * S + (i % (K / W)) * W;
#pragma unroll
            for (int t = 0; t < W; ++t) d[t] = v[u][t];
          }
        }
      }
    } else {
      copy_in<NT>(st, S, src, K, K, np, tid, false);
    }
    __syncthreads();
    T g[3] = {T(0), T(0), T(0)};
    vjp_parts<T, LT, NORM, E3, DS>(std::make_integer_sequence<int, DS>{}, h, pt, st,
                               (lane < np ? lane : np - 1) * S, P.conv, g);
    if constexpr (DS > 1) {
      if (h > 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) sacc[((h - 1) * 3 + a) * kWave + lane] = g[a];
      }
      __syncthreads();
      if (h == 0) {
#pragma unroll
        for (int w = 0; w < DS - 1; ++w)
#pragma unroll
          for (int a = 0; a < 3; ++a) g[a] += sacc[(w * 3 + a) * kWave + lane];
      }
    }
    if (h == 0 && lane < np) {
      T* o = static_cast<T*>(P.gxyz) + (p0 + lane) * 3;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        // e3nn: the points are (z, x, y), so d/dx is the second axis' sum
        const T v = E3 ? g[(a + 1) % 3] : g[a];
        o[a] = NORM ? v * pt.inv_r : v;
      }
    }
    if (tile + gridDim.x < (P.n + kWave - 1) / kWave) __syncthreads();  // another tile: every read of this one is done
  }
}

}  // namespace sph
