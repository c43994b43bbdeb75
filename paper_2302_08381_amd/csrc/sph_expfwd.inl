// Radial expansion for compile-time degrees (l_max <= 12) and up to 16 channels:
//   c[e, n, l^2+l+m] = sum over the points j of environment e of
//                      R[j, l, n] * Y_l^m(x_j)
// (sph_expand.inl holds the kernel for the rest).
//
// A block takes chunks of up to 64 (or 32) consecutive points.  Its waves
// split the degrees to write the chunk's harmonics into an LDS tile, the
// radial rows are copied next to it, and the chunk is contracted by items: an
// item is the two columns +-m of a degree times CW channels, so a point costs
// its thread two harmonics and CW radial values from LDS for 2 CW
// multiply-adds (items of one column are bound by those reads).  The threads
// form several parts, each a full set of items that takes every parts-th
// point; a thread's sums stay in registers from chunk to chunk until its
// environment ends, when the parts' sums meet in LDS, in a fixed order, and
// leave as contiguous rows of c.  The walk through the environments looks at
// 64 offsets at a time; a chunk runs through as many environments as it holds,
// and the next chunk's radial rows are in flight during the arithmetic.
//
// Measured, 1.36e6 points in 20 000 environments, against one column per item,
// two environments per chunk and sums through LDS between chunks: float 8
// channels l_max 3 65 -> 45 us, l_max 6 202 -> 92, l_max 8 188 -> 130 (3.5
// TB/s of 0.46 GB), l_max 12 325 -> 232; 16 channels l_max 8 439 -> 210; 5
// channels l_max 8 232 -> 137; double 4 channels l_max 6 180 -> 108, 8
// channels l_max 8 363 -> 281; 136 000 points in 2000 environments, double 5
// channels l_max 6 48 -> 24.  What is left is arithmetic and LDS: the
// harmonics take about a third of a chunk, the contraction most of the rest.
#pragma once

#include "sph_expand.inl"

namespace sph {


// Shape of the kernel for l_max LT, NG groups of CW channels and WV waves.
template <typename T, int LT, int CW, int NG, int WV>
struct ExpFwd {
  static constexpr int K = (LT + 1) * (LT + 1);
  static constexpr int NP = CW * NG;                             // padded channels
  static constexpr int pairs = (LT + 1) * (LT + 2) / 2;          // (l, m >= 0)
  static constexpr int items = pairs * NG;
  static constexpr int SY = K | 1;                               // odd: conflict-free column reads
  static constexpr int RS = (LT + 1) * NP;
  static constexpr size_t lds(int points, int parts) {
    return sizeof(T) * (static_cast<size_t>((points * SY + 3) / 4 * 4) + static_cast<size_t>(points) * RS +
                        static_cast<size_t>(parts) * NP * K);
  }
  static constexpr int max_parts = kWave * WV / items < 16 ? kWave * WV / items : 16;
  // The largest number of parts (up to a quarter fewer than there are threads
  // for) and 64 points that let sixteen waves, or the most down to three (in
  // double, whose registers allow three, two) blocks share a CU's LDS; else 32
  // points.  Against 32
  // points: float 8 channels l_max 6 92 and 123 us, l_max 8 130 and 142;
  // double 5 channels l_max 6 26 and 34.  Against 64 points where fewer blocks
  // would fit: float 16 channels l_max 12 224 and 340, double 8 channels l_max
  // 8 281 and 350.
  static constexpr int shape() {
    for (int blocks = 16 / WV; blocks >= (sizeof(T) == 8 ? 2 : 3); --blocks)
      for (int p = max_parts; 4 * p >= 3 * max_parts; --p)
        if (lds(64, p) * blocks <= 160 * 1024) return 64 + 1024 * p;
    return 32 + 1024 * max_parts;
  }
  static constexpr int parts = shape() / 1024;
  static constexpr int CP = shape() % 1024;
  static constexpr size_t lds_bytes = lds(CP, parts);
  static_assert(parts >= 1, "a part fits the block");
};

// Harmonics of degrees [LA, LB) of one point into its LDS row.
template <typename T, bool NORM, int LA, int LB>
__device__ __forceinline__ void expfwd_rows(const Point<T>& pt, T* row) {
  if constexpr (LA < LB) {
    constexpr int MM = LB - 1;
    constexpr T kIS2 = T(kInvSqrt2d);
    T c[MM + 1], s[MM + 1];
    c[0] = T(1);
    s[0] = T(0);
#pragma unroll
    for (int m = 1; m <= MM; ++m) {
      s[m] = pt.ex * s[m - 1] + pt.ey * c[m - 1];
      c[m] = pt.ex * c[m - 1] - pt.ey * s[m - 1];
    }
    T cur[MM + 3];
#pragma unroll
    for (int l = LA; l < LB; ++l) {
      q_row<T, MM>(l, pt.ez, pt.rxy2, cur);
      const int k0 = l * l + l;
      row[k0] = cur[0] * kIS2;
#pragma unroll
      for (int m = 1; m <= MM; ++m) {
        if (m > l) continue;  // no early exit: keeps the loop fully unrolled
        row[k0 + m] = cur[m] * c[m];
        row[k0 - m] = cur[m] * s[m];
      }
    }
  }
}

template <typename T, int LT, bool NORM, int WV, int... Hs>
__device__ __forceinline__ void expfwd_parts(std::integer_sequence<int, Hs...>, int h, const Point<T>& pt, T* row) {
  ((h == Hs ? expfwd_rows<T, NORM, degree_split(LT, WV, Hs), degree_split(LT, WV, Hs + 1)>(pt, row)
            : void()),
   ...);
}

// Radial accesses in flight per thread for the next chunk: all of it where
// that takes six 16-byte vectors (double on two waves, whose blocks are few:
// ten), else so many.
template <typename T, int WV>
constexpr int expfwd_batch(int all, int ew) {
  const int most = (sizeof(T) == 8 && WV == 2 ? 10 : 6) * (Vec16<T>::n / ew);
  return all < most ? all : most;
}

template <typename T, int LT, bool NORM, int CW, int NG, int WV, bool VEC>
__global__ __launch_bounds__(kWave * WV) void k_expfwd(ExpandParams P) {
  using F = ExpFwd<T, LT, CW, NG, WV>;
  using V = typename Vec16<T>::type;
  constexpr int W = Vec16<T>::n;
  // an item's channels as the widest vectors that divide them
  constexpr int CV = CW % W == 0 ? W : 2;
  typedef T C __attribute__((ext_vector_type(CV)));
  constexpr int NT = kWave * WV;
  constexpr int L = LT, K = F::K, NP = F::NP, SY = F::SY, RS = F::RS, CP = F::CP;
  extern __shared__ __align__(16) unsigned char smem[];
  T* sY = reinterpret_cast<T*>(smem);
  T* sR = sY + (CP * SY + 3) / 4 * 4;
  T* sP = sR + CP * RS;
  const int tid = threadIdx.x, lane = tid % kWave, h = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int NM = P.n_max;
  const T* xyz = static_cast<const T*>(P.xyz);
  const T* R = static_cast<const T*>(P.R);
  T* cout = static_cast<T*>(P.c);
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
  // lane i: where environment e + i ends relative to j0, at most CP + 1
  auto window = [&]() {
    const int64_t i = e + 1 + lane;
    const int64_t d = offset(i < e_end ? i : e_end) - j0;
    return static_cast<int>(d < 0 ? 0 : (d > CP ? CP + 1 : d));
  };
  auto rows_left = [&](int64_t j) {  // (none where inconsistent offsets end before j)
    const int64_t d = j_end - j;
    return __builtin_amdgcn_readfirstlane(static_cast<int>(d < 0 ? 0 : (d < CP ? d : CP)));
  };
  // The radial rows of a chunk: global [cnt][L+1][NM] to LDS rows [L+1][NP].
  // VEC (NM == NP, R 16-byte aligned): a straight copy of vectors; else
  // element by element, (row, channel) of a thread's elements by counters.
  using E = std::conditional_t<VEC, V, T>;
  constexpr int EW = VEC ? W : 1;
  constexpr int NB = expfwd_batch<T, WV>((CP * RS / EW + NT - 1) / NT, EW);
  const int row_len = (L + 1) * (VEC ? NP : NM);
  const int crow = VEC ? 0 : tid / NM, cch = VEC ? 0 : tid - crow * NM;
  const int qs = VEC ? 0 : NT / NM, rq = VEC ? 0 : NT - qs * NM;
  E rv[NB];
  T px = T(0), py = T(0), pz = T(0);
  auto load_rows = [&](int64_t j, int cnt, int from) {
    const E* gp = reinterpret_cast<const E*>(R + j * row_len);
    const int ne = cnt * row_len / EW;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int i = from + tid + u * NT;
      if (i < ne) rv[u] = __builtin_nontemporal_load(gp + i);
    }
  };
  int srow = 0, sch = 0;
  auto store_rows = [&](int cnt, int from) {
    const int ne = cnt * row_len / EW;
    E* d = reinterpret_cast<E*>(sR);
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int i = from + tid + u * NT;
      if constexpr (VEC) {
        if (i < ne) d[i] = rv[u];
      } else {
        if (i < ne) d[srow * NP + sch] = rv[u];
        srow += qs;
        sch += rq;
        if (sch >= NM) {
          sch -= NM;
          ++srow;
        }
      }
    }
  };
  auto load_point = [&](int64_t j, int cnt) {
    const T* q = xyz + (j + (lane < cnt ? lane : cnt - 1)) * 3;
    px = q[0];
    py = q[1];
    pz = q[2];
  };
  auto zero_env = [&](int64_t ee) {
    T* ce = cout + ee * NM * K;
    for (int i = tid; i < NM * K; i += NT) ce[i] = T(0);
  };

  // this thread's item: (l, m) and channel group, and its part
  const int part = tid / F::items, it = tid - part * F::items;
  const bool on = part < F::parts;
  const int cg = on ? it / F::pairs : 0;
  const int pi = on ? it - cg * F::pairs : 0;
  int il = static_cast<int>((sqrtf(8.0f * static_cast<float>(pi) + 1.0f) - 1.0f) * 0.5f);
  il += (il + 1) * (il + 2) / 2 <= pi ? 1 : 0;
  il -= il * (il + 1) / 2 > pi ? 1 : 0;
  const int im = pi - il * (il + 1) / 2;
  const int kp = il * il + il + im, km = il * il + il - im;
  const int ro = il * NP + cg * CW;
  T ap[CW], am[CW];
#pragma unroll
  for (int u = 0; u < CW; ++u) ap[u] = am[u] = T(0);

  if constexpr (!VEC) {  // the padding channels stay zero
    for (int i = tid; i < CP * RS; i += NT) sR[i] = T(0);
    __syncthreads();
  }
  int wend = window();
  int left = rows_left(j0);
  if (left > 0) {
    load_rows(j0, left, 0);
    load_point(j0, left);
  }
  for (;;) {
    // the chunk: up to CP points of the window's environments
    const int wlast = __builtin_amdgcn_readlane(wend, kWave - 1);
    const int cnt = wlast < CP ? wlast : CP;
    const int before = __shfl_up(wend, 1);
    const unsigned long long full = __ballot(wend > (lane == 0 ? 0 : before));  // not empty
    const int64_t we = e;  // the window's first environment
    // environments done with this chunk: `done` of the window
    const unsigned long long reach = __ballot(wend >= cnt);
    const int kl = cnt == 0 ? kWave - 1 : __builtin_ctzll(reach);  // holds the last point
    const bool inside = cnt > 0 && __builtin_amdgcn_readlane(wend, kl) > cnt;
    int done = inside ? kl : kl + 1;
    if (done > e_end - e) done = static_cast<int>(e_end - e);
    // the empty ones among them
    for (unsigned long long z = ~full & (done >= kWave ? ~0ull : (1ull << done) - 1); z != 0; z &= z - 1)
      zero_env(we + __builtin_ctzll(z));
    if (cnt > 0) {
      srow = crow;
      sch = cch;
      store_rows(cnt, 0);
#pragma unroll 1
      for (int from = NB * NT; from < cnt * row_len / EW; from += NB * NT) {
        load_rows(j0, cnt, from);
        store_rows(cnt, from);
      }
    }
    const T x = px, y = py, z = pz;
    const int wcur = wend;
    // the next chunk's loads, in flight during this one's arithmetic
    e += done;
    j0 += cnt;
    const bool more = e < e_end;
    if (more) {
      wend = window();
      left = rows_left(j0);
      if (left > 0) {
        load_rows(j0, left, 0);
        load_point(j0, left);
      }
    }
    if (cnt > 0) {
      if (lane < cnt) {
        const Point<T> pt = make_point<T, NORM>(x, y, z);
        expfwd_parts<T, LT, NORM, WV>(std::make_integer_sequence<int, WV>{}, h, pt, sY + lane * SY);
      }
      __syncthreads();
      // environment by environment
      int s = 0;
      unsigned long long todo = full;
      while (s < cnt && todo != 0) {
        const int k = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int v = __builtin_amdgcn_readlane(wcur, k);
        const int t = v < cnt ? v : cnt;
        if (on) {
          const T* yp = sY + kp;
          const T* ym = sY + km;
          const T* rp = sR + ro;
#pragma unroll 2
          for (int j = s + part; j < t; j += F::parts) {
            const T vp = yp[j * SY], vm = ym[j * SY];
            const C* r = reinterpret_cast<const C*>(rp + j * RS);
#pragma unroll
            for (int a = 0; a < CW / CV; ++a) {
              const C q = r[a];
#pragma unroll
              for (int u = 0; u < CV; ++u) {
                ap[a * CV + u] += q[u] * vp;
                am[a * CV + u] += q[u] * vm;
              }
            }
          }
        }
        s = t > s ? t : s;
        if (v <= cnt) {  // the environment ends here: the parts' sums, in order
          if (on) {
            T* d = sP + part * (NP * K) + cg * CW * K;
#pragma unroll
            for (int u = 0; u < CW; ++u) {
              d[u * K + kp] = ap[u];
              if (im > 0) d[u * K + km] = am[u];
              ap[u] = am[u] = T(0);
            }
          }
          __syncthreads();
          T* ce = cout + (we + k) * NM * K;
          for (int i = tid; i < NM * K; i += NT) {
            T v0 = sP[i];
#pragma unroll
            for (int q = 1; q < F::parts; ++q) v0 += sP[q * (NP * K) + i];
            ce[i] = v0;
          }
          __syncthreads();  // sP may be written again
        }
      }
    }
    if (!more) break;
    __syncthreads();  // every read of the tiles is done
  }
}

}  // namespace sph
