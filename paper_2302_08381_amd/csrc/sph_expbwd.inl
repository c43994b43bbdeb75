// Backward of the radial expansion for compile-time degrees (l_max <= 12, but
// double with 9..16 channels <= 6); sph_expand.inl holds the run-time-degree kernel
// and states the sums:
//   grad_R[j, l, n] = sum_m G[e, n, l^2+l+m] Y_l^m(x_j)
//   grad_xyz[j, a]  = sum_k gY[j, k] dY_k/dx_a(x_j),
//                     gY[j, k] = sum_n G[e, n, k] R[j, l(k), n]
//
// A block takes chunks of 64 consecutive points, one lane per point, and
// splits the degrees between its DS waves: the waves share the chunk's LDS
// tile of radial rows and the G of its environments, so a CU holds twice (or
// four times) the waves that one lane set per tile would give it, and every
// wave's unrolled degrees have literal coefficients.  A chunk runs through up
// to kExpBwdSlices environments; their G wait in as many LDS slices
// ([column][channel], read as 16-byte vectors).  Radial rows arrive by
// coalesced copies, the next chunk's in flight during this one's arithmetic,
// and grad_R leaves through the same slots.
//
// Bound by its copies and the walk: without the arithmetic the same kernel
// takes 195 us of its 207 at l_max 8 (float, 8 channels, 20 000 environments
// of 8..128 points, 4.2 TB/s of the bytes it cannot avoid).  Against one wave
// per lane set with run-time degrees: l_max 8 385 -> 207 us, l_max 12 785 ->
// 340, l_max 3 97 -> 72; 5 channels l_max 8 582 -> 254; double l_max 8 686 ->
// 490.
#pragma once

#include "sph_expand.inl"

namespace sph {

constexpr int kExpBwdPoints = kWave;  // points per chunk

// The copy back, by expand_tile_in's walk.
template <typename T, int NPC, int NT, int MODE>
__device__ __forceinline__ void expand_tile_out(const T* __restrict__ sR, int RS, T* __restrict__ dst, int cnt,
                                                int L, int NM, int gl) {
  constexpr int U = MODE == 1 ? Vec16<T>::n : 1;
  using E = std::conditional_t<U == 1, T, typename Vec16<T>::type>;
  constexpr int SL = NPC / U;
  constexpr int RPS = NT / SL;
  const int n = (gl % SL) * U, L1 = L + 1, rows = cnt * L1;
  int p = (gl / SL) / L1, l = gl / SL - p * L1;
  const int qs = RPS / L1, rq = RPS - qs * L1;
  if (n < NM) {
    for (int r = gl / SL; r < rows; r += RPS) {
      *reinterpret_cast<E*>(dst + r * NM + n) = *reinterpret_cast<const E*>(sR + p * RS + l * NPC + n);
      p += qs;
      l += rq;
      if (l >= L1) {
        l -= L1;
        ++p;
      }
    }
  }
}

// Radial vectors in flight per thread for the next chunk (an l_max 8 tile of
// 8 channels takes 9 in float on two waves, 9 in double on four).
constexpr int kExpBwdBatch = 10;

// Whether whole-vector rows take the VEC kernel: not float with 16 channels
// past l_max 4, where its prefetched rows make the unrolled degrees spill
// (10 000 environments, l_max 9: 602 us against 344 with the general
// copies).
template <typename T>
constexpr bool expbwd_vec(int LT, int npc) {
  return !(sizeof(T) == 4 && npc == 16 && LT > 4);
}

// Degrees [LA, LB) of one point: sG its environment's G, row its radial row
// in LDS ([degree][NPC]), which the degree's grad_R replaces.  Adds to g.
template <typename T, bool NORM, int NPC, int LA, int LB>
__device__ __forceinline__ void expbwd_degrees(const Point<T>& pt, const T* st, int og, int orow, T (&g)[3],
                                               T* stw) {
  using V = typename Vec16<T>::type;
  constexpr int W = Vec16<T>::n;
  constexpr int NV = NPC / W;
  constexpr int MM = LB - 1;
  constexpr T kIS2 = T(kInvSqrt2d);
  const CoefTable<T>& C = coef<T>();
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
  T x0 = T(0), y0 = T(0), z0 = T(0);
  // G of one order's columns k0 + m (gp) and k0 - m (gm), read one order
  // ahead: a fence after each order keeps the compiler from reading further
  // ahead, which spilled
  V gp[NV], gm[NV];
  auto read_g = [&](int l, int m, V (&p)[NV], V (&q)[NV]) {
#pragma unroll
    for (int h = 0; h < NV; ++h) {
      p[h] = *reinterpret_cast<const V*>(st + og + (l * l + l + m) * NPC + h * W);
      if (m > 0) q[h] = *reinterpret_cast<const V*>(st + og + (l * l + l - m) * NPC + h * W);
    }
  };
  read_g(LA, 0, gp, gm);
#pragma unroll
  for (int l = LA; l < LB; ++l) {
    q_row<T, MM>(l, ez, pt.rxy2, cur);
    T r[NPC], acc[NPC];
#pragma unroll
    for (int h = 0; h < NV; ++h) {
      const V v = *reinterpret_cast<const V*>(st + orow + l * NPC + h * W);
#pragma unroll
      for (int u = 0; u < W; ++u) {
        r[h * W + u] = v[u];
        acc[h * W + u] = T(0);
      }
    }
    // a column of value Y and derivatives (dx, dy, dz) up to the chain rule's 1/r
    auto col = [&](const V (&gv)[NV], T Y, T dx, T dy, T dz) {
      T gy = T(0);
#pragma unroll
      for (int n = 0; n < NPC; ++n) {
        gy += gv[n / W][n % W] * r[n];
        acc[n] += gv[n / W][n % W] * Y;
      }
      x0 += gy * dx;
      y0 += gy * dy;
      z0 += gy * dz;
    };
    const T lz = T(l) * ez;
#pragma unroll
    for (int m = 0; m <= MM; ++m) {
      if (m > l) continue;  // no early exit: keeps the loop fully unrolled
      V np[NV], nm[NV];
      if (m < l)
        read_g(l, m + 1, np, nm);
      else if (l + 1 < LB)
        read_g(l + 1, 0, np, nm);
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
        col(gp, q * kIS2, dx * kIS2, dy * kIS2, e * kIS2);
      } else {
        const T qc = q * mc[m], qs = q * ms[m];
        col(gp, q * c[m], dx * c[m] + qc, dy * c[m] - qs, e * c[m]);
        col(gm, q * s[m], dx * s[m] + qs, dy * s[m] + qc, e * s[m]);
      }
#pragma unroll
      for (int h = 0; h < NV; ++h) {
        gp[h] = np[h];
        gm[h] = nm[h];
      }
      asm volatile("" : "+v"(og), "+v"(x0), "+v"(y0), "+v"(z0));
    }
#pragma unroll
    for (int h = 0; h < NV; ++h) {
      V v;
#pragma unroll
      for (int u = 0; u < W; ++u) v[u] = acc[h * W + u];
      *reinterpret_cast<V*>(stw + orow + l * NPC + h * W) = v;
    }
    copy_row<T, MM>(l, cur, prev);
    // the next degree starts after this one (as in vjp_degrees)
    asm volatile("" : "+v"(ez), "+v"(og), "+v"(orow), "+v"(x0), "+v"(y0), "+v"(z0));
  }
  g[0] += x0;
  g[1] += y0;
  g[2] += z0;
}

template <typename T, int LT, bool NORM, int NPC, int DS, int... Hs>
__device__ __forceinline__ void expbwd_parts(std::integer_sequence<int, Hs...>, int h, const Point<T>& pt, T* st,
                                             int og, int orow, T (&g)[3]) {
  ((h == Hs ? expbwd_degrees<T, NORM, NPC, degree_split(LT, DS, Hs), degree_split(LT, DS, Hs + 1)>(pt, st, og, orow,
                                                                                                 g, st)
            : void()),
   ...);
}

// Waves per SIMD that the registers are bounded for.
template <typename T>
constexpr int expbwd_occupancy() {
  return sizeof(T) == 4 ? 2 : 1;
}

// Dynamic LDS: expbwd_lds_bytes.  P.slices: environments per chunk.
// VEC: every padded channel is present and both radial arrays are 16-byte
// aligned, so rows are whole vectors; otherwise the general copies (their
// addresses kept out of the loop's registers).  One kernel with both paths
// ran 206 -> 247 us at l_max 8.
template <typename T, int LT, bool NORM, int NPC, int DS, bool VEC>
__global__ __launch_bounds__(kWave * DS) __attribute__((amdgpu_waves_per_eu(expbwd_occupancy<T>()))) void k_expbwd(ExpandBwdParams P) {
  using V = typename Vec16<T>::type;
  constexpr int W = Vec16<T>::n;
  constexpr int NT = kWave * DS;
  constexpr int L = LT, K = (L + 1) * (L + 1);
  constexpr int RS = expand_bwd_row_stride<T>(L, NPC);
  constexpr int CP = kExpBwdPoints;
  constexpr int MS = kExpBwdSlices;
  constexpr int RV = (L + 1) * NPC / W;  // vectors of a padded row
  extern __shared__ __align__(16) unsigned char smem[];
  T* st = reinterpret_cast<T*>(smem);  // the radial tile, then the G slices, then the partial sums
  const int NS = P.slices;
  constexpr int oG = CP * RS;
  constexpr int slice = K * NPC;
  T* sacc = st + oG + NS * slice;
  const int tid = threadIdx.x, lane = tid % kWave, h = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int NM = P.n_max;
  const T* xyz = static_cast<const T*>(P.xyz);
  const T* R = static_cast<const T*>(P.R);
  const T* gc = static_cast<const T*>(P.gc);
  T* gxyz = static_cast<T*>(P.gxyz);
  T* gR = static_cast<T*>(P.gR);
  // the channels fill whole vectors short of the padding
  const bool vpart = !VEC && NM % W == 0 && aligned16(R) && (gR == nullptr || aligned16(gR));

  if (P.status != nullptr && blockIdx.x == 0 && tid < kWave) {
    bool ok = true;
    for (int64_t i = lane; i < P.n_env; i += kWave) ok = ok && (P.offsets[i] <= P.offsets[i + 1]);
    if (lane == 0) ok = ok && P.offsets[0] == 0 && P.offsets[P.n_env] == P.n;
    const bool all_ok = __all(ok);
    if (lane == 0) P.status[0] = all_ok ? 0 : 4 /* SPH_ERR_OFFSETS */;
  }

  int64_t e, e_end;  // this block's environments
  block_share(P.offsets, P.n_env, P.n, lane, e, e_end);
  if (e >= e_end) return;
  // offsets clamped into [0, n], so that inconsistent ones (reported through
  // the status word) never index out of bounds
  auto offset = [&](int64_t i) {
    const int64_t o = P.offsets[i];
    return o < 0 ? int64_t(0) : (o > P.n ? P.n : o);
  };
  int64_t j0 = uniform64(offset(e));
  const int64_t j_end = uniform64(offset(e_end));
  // The walk looks at 64 environments at once: lane i holds where environment
  // e + i ends relative to j0, at most CP + 1.
  auto window = [&]() {
    const int64_t i = e + 1 + lane;
    const int64_t d = offset(i < e_end ? i : e_end) - j0;
    return static_cast<int>(d < 0 ? 0 : (d > CP ? CP + 1 : d));
  };
  // this thread's vectors of a chunk's radial rows (VEC), and its point;
  // cnt: rows that exist past j0, at most CP
  V rv[kExpBwdBatch];
  T px = T(0), py = T(0), pz = T(0);
  auto rows_left = [&](int64_t j) {  // (none where inconsistent offsets end before j)
    const int64_t d = j_end - j;
    return static_cast<int>(d < 0 ? 0 : (d < CP ? d : CP));
  };
  // Vectors from .. of the tile's rows in global order; vector i of the block
  // of rows is vector i % RV of LDS row i / RV, walked with running counters
  // (one division).  f(u, i, LDS element).
  auto each_vector = [&](int nv, int from, int ti, auto&& f) {
    const int i0 = from + ti;
    int c = i0 % RV, o = i0 / RV * RS + c * W;
    constexpr int rq = NT % RV, so = NT / RV * RS + rq * W;
#pragma unroll
    for (int u = 0; u < kExpBwdBatch; ++u) {
      if (u * NT >= CP * RV) break;  // a whole chunk's rows
      if (i0 + u * NT < nv) f(u, i0 + u * NT, o);
      o += so;
      c += rq;
      if (c >= RV) {
        c -= RV;
        o += RS - RV * W;
      }
    }
  };
  auto load_rows = [&](int64_t j, int cnt, int from, int ti) {
    const V* gp = reinterpret_cast<const V*>(R + j * (L + 1) * NM);
    const int i0 = from + ti, nv = cnt * RV;
#pragma unroll
    for (int u = 0; u < kExpBwdBatch; ++u)
      if (u * NT < CP * RV && i0 + u * NT < nv) rv[u] = __builtin_nontemporal_load(gp + i0 + u * NT);
  };
  auto store_rows = [&](int cnt, int from, int ti) {
    each_vector(cnt * RV, from, ti, [&](int u, int, int o) { *reinterpret_cast<V*>(st + o) = rv[u]; });
  };
  auto rows_out = [&](T* dst, int cnt, int ti) {
    V* gp = reinterpret_cast<V*>(dst);
#pragma unroll 1
    for (int from = 0; from < cnt * RV; from += kExpBwdBatch * NT)
      each_vector(cnt * RV, from, ti, [&](int, int i, int o) { gp[i] = *reinterpret_cast<const V*>(st + o); });
  };
  auto load_point = [&](int64_t j, int cnt) {
    const T* q = xyz + (j + (lane < cnt ? lane : cnt - 1)) * 3;
    px = q[0];
    py = q[1];
    pz = q[2];
  };

  int slot = 0;           // the LDS slice of the chunk's first environment
  bool resident = false;  // whose G is there already
  int wend = window();
  {
    const int left = __builtin_amdgcn_readfirstlane(rows_left(j0));
    if (left <= 0) return;  // only empty environments
    if constexpr (VEC) load_rows(j0, left, 0, tid);
    load_point(j0, left);
  }
  for (;;) {
    // general copies: the thread's index, opaque to the compiler, which would
    // keep the addresses of every copy below in registers from one chunk to
    // the next
    int ti = tid;
    if constexpr (!VEC) asm volatile("" : "+v"(ti));
    // The chunk: the first NS non-empty environments of the window, up to CP
    // points; the i-th is e + de[i] and ends at point end[i] of the chunk.
    int de[MS], end[MS], cnt = 0, ne = 0, last = 0;
    {
      const int before = __shfl_up(wend, 1);
      unsigned long long mask = __ballot(wend > (lane == 0 ? 0 : before));
#pragma unroll
      for (int i = 0; i < MS; ++i) {
        de[i] = 0;
        end[i] = CP;
        if (i < NS && mask != 0 && cnt < CP) {
          const int k = __builtin_ctzll(mask);
          const int v = __builtin_amdgcn_readlane(wend, k);
          mask &= mask - 1;
          de[i] = k;
          last = v;
          if (v > cnt) cnt = v > CP ? CP : v;  // (not more only with inconsistent offsets)
          end[i] = cnt;
          ne = i + 1;
        }
      }
    }
    if (ne == 0) {  // 64 empty environments
      e += kWave;
      resident = false;
      if (e >= e_end) break;
      wend = window();
      continue;
    }
    // G of the chunk's new environments, [n][k] -> [k][n], padding channels
    // zero: one thread per column, its channels loaded together
    const int i0 = resident ? 1 : 0;
#pragma unroll 1
    for (int q = ti; q < (ne - i0) * K; q += NT) {
      const int i = i0 + q / K, k = q % K;
      int d = de[0];
#pragma unroll
      for (int a = 1; a < MS; ++a) d = i == a ? de[a] : d;
      const T* ge = gc + (e + d) * NM * K + k;
      T v[NPC];
#pragma unroll
      for (int n = 0; n < NPC; ++n) v[n] = n < NM ? ge[n * K] : T(0);
      int sl = slot + i;
      sl = sl >= NS ? sl - NS : sl;
      V* dst = reinterpret_cast<V*>(st + oG + sl * slice + k * NPC);
#pragma unroll
      for (int a = 0; a < NPC / W; ++a) {
        V w;
#pragma unroll
        for (int u = 0; u < W; ++u) w[u] = v[a * W + u];
        dst[a] = w;
      }
    }
    if constexpr (VEC) {
      store_rows(cnt, 0, ti);
#pragma unroll 1
      for (int from = kExpBwdBatch * NT; from < cnt * RV; from += kExpBwdBatch * NT) {
        load_rows(j0, cnt, from, ti);
        store_rows(cnt, from, ti);
      }
    } else if (vpart) {
      expand_tile_in<T, NPC, NT, 1>(st, RS, R + j0 * (L + 1) * NM, cnt, L, NM, ti);
    } else {
      expand_tile_in<T, NPC, NT, 0>(st, RS, R + j0 * (L + 1) * NM, cnt, L, NM, ti);
    }
    const T x = px, y = py, z = pz;
    // the next chunk's loads, in flight during this one's arithmetic
    const int64_t jc = j0;
    const bool inside = last > cnt;  // the last environment goes on
    int dl = de[0];
#pragma unroll
    for (int a = 1; a < MS; ++a) dl = ne > a ? de[a] : dl;
    e += dl + (inside ? 0 : 1);
    j0 += cnt;
    const int left = __builtin_amdgcn_readfirstlane(e < e_end ? rows_left(j0) : 0);
    if (left > 0) {
      wend = window();
      if constexpr (VEC) load_rows(j0, left, 0, ti);
      load_point(j0, left);
    }
    __syncthreads();
    T gs[3] = {T(0), T(0), T(0)};
    const Point<T> pt = make_point<T, NORM>(x, y, z);
    {
      // this lane's environment among the chunk's (lanes past the chunk's
      // points work on whatever the tile holds; nothing of theirs is stored)
      int i = 0;
#pragma unroll
      for (int a = 0; a < MS - 1; ++a) i += (a + 1 < ne && lane >= end[a]) ? 1 : 0;
      int sl = slot + i;
      sl = sl >= NS ? sl - NS : sl;
      expbwd_parts<T, LT, NORM, NPC, DS>(std::make_integer_sequence<int, DS>{}, h, pt, st, oG + sl * slice, lane * RS,
                                         gs);
    }
    if (h > 0) {
#pragma unroll
      for (int a = 0; a < 3; ++a) sacc[((h - 1) * 3 + a) * kWave + lane] = gs[a];
    }
    __syncthreads();
    if (h == 0 && gxyz != nullptr && lane < cnt) {
      T* o = gxyz + (jc + lane) * 3;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        T v = gs[a];
#pragma unroll
        for (int w = 0; w < DS - 1; ++w) v += sacc[(w * 3 + a) * kWave + lane];
        o[a] = NORM ? v * pt.inv_r : v;
      }
    }
    if constexpr (!VEC) asm volatile("" : "+v"(ti));
    if (gR != nullptr) {
      T* dst = gR + jc * (L + 1) * NM;
      if constexpr (VEC)
        rows_out(dst, cnt, ti);
      else if (vpart)
        expand_tile_out<T, NPC, NT, 1>(st, RS, dst, cnt, L, NM, ti);
      else
        expand_tile_out<T, NPC, NT, 0>(st, RS, dst, cnt, L, NM, ti);
    }
    if (left <= 0) break;
    __syncthreads();  // every read of the tile, the slices and the sums is done
    slot += inside ? ne - 1 : ne;
    slot = slot >= NS ? slot - NS : slot;
    resident = inside;
  }
}

}  // namespace sph
