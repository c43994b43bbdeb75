// Explicit second derivatives: d2Y[i][a][b][k] = d^2 Y_k / (dx_a dx_b) at
// point i, the full symmetric 3x3 block of every column (Sec. II: the
// Cartesian recursion gives derivatives of any order by applying Eq.
// iter-deri again).
//
// Mapping: one lane per (point, order), or two, one per sign of the order, in
// waves of their own.  A lane walks the degrees l = m .. l_max upward at fixed
// order with the recursion of OrdChain carried one derivative further:
// p_l = Qt_l^m / N_l^m, e = 2 dp/d(rho^2), w = 2 de/d(rho^2), and along z
// dp_l/dz = (l-m) p_{l-1}.  With T = N e, W = N w, V = N (l-m) e_{l-1},
// U = N (l-m)(l-1-m) p_{l-2},
//   H(Qt) = [ T + x^2 W   x y W       x V ]
//           [             T + y^2 W   y V ]
//           [                         U   ]
// and with the order's factor t = c_m or s_m the six unique entries of a
// column are
//   H(Qt t) = t H(Qt) + grad Qt grad t' + grad t grad Qt' + Qt H(t).
// For the normalised harmonics Y(x) = Yt(u), u = x / r, with g = grad Yt(u),
//   H Y = [ H Yt - l (u s' + s u') - l Yt 1 ] / r^2,  s = g - (l+2)/2 Yt u.
// The entries go into an LDS tile laid out like the global block
// [points][3][3][K] and leave as 16-byte stores.
//
// The tile decides how many points a CU holds at once (1.8 KB each at l_max 6
// in float), so the orders and signs are what fills its waves; a lane per row
// of the 3x3 block forms each off-diagonal entry twice and the shared factors
// three times.  Measured against that, 1e6 points: float l_max 3 124 -> 106 us,
// l_max 6 392 -> 300 (5.9 TB/s of stores), l_max 8 (500 000) 511 -> 250, l_max
// 12 (300 000) 1242 -> 340; double l_max 4 (500 000) 192 -> 158, l_max 8 (300
// 000) 827 -> 300; l_max 32 float (30 000) 1395 -> 398, double (10 000) 1156 ->
// 316.  What is left up to l_max 12 is close to the stores, beside about 90
// operations per column, of which the lanes below their order waste a quarter;
// past it the few waves that the tile leaves.  Error against double, float l_max 6 / 12: 5e-7 / 6e-7
// of a point's largest entry (1.6e-6 / 2e-6).
#pragma once

#include "sph_ord.inl"

namespace sph {

// LDS elements of a tile of `points` Hessians.  A point's nine rows take a
// stride that is padded by one 16-byte vector where it would bring the lanes of
// one order to few banks: float l_max + 1 a multiple of 4 (9 K is then a
// multiple of 16; else it is odd, or 4 times an odd number, which keeps 16
// points and 4 orders apart), double odd l_max.
template <typename T>
__host__ __device__ constexpr int hess_pad(int L) {
  if (sizeof(T) == 4) return (L + 1) % 4 == 0 ? 4 : 0;
  return (L & 1) != 0 ? 2 : 0;
}
template <typename T>
__host__ __device__ constexpr size_t hess_lds_bytes(int L, int points) {
  return sizeof(T) * static_cast<size_t>(ord_block<T>(points * (9 * (L + 1) * (L + 1) + hess_pad<T>(L))));
}

// Waves per order (one, or two for the two signs) and points per tile: the
// signs apart from l_max 6 (float l_max 5 255 us against 223 together, l_max 6
// 308 and 310, l_max 8 260 and 270, l_max 12 359 and 406); the most points of
// one wave, or two with the signs apart, whose tile leaves three blocks in a
// CU's LDS and whose lanes fill three quarters of their waves (float l_max 6
// 18 points 308 us, 14 339; l_max 12 8 points 359, 9 408 and 4 397; double
// l_max 7 8 points 242, 11 283); where no number does, the most that fit.
constexpr int hess_split(int L) { return L >= 6 ? 2 : 1; }
template <typename T>
constexpr int hess_points(int L) {
  const int lanes = 64 * hess_split(L);
  int most = 1;
  for (int p = 2; p * (L + 1) <= lanes && hess_lds_bytes<T>(L, p) <= 53 * 1024; ++p) most = p;
  for (int p = most; p >= 1; --p) {
    const int used = p * (L + 1);
    if (4 * used >= 3 * ((used + 63) / 64 * 64)) return p;
  }
  return most;
}

// LT: l_max at compile time, or -1 (P.L).  P.tile points per block; SP waves
// per order of P.tile (l_max + 1) lanes, rounded up to whole waves.  Dynamic
// LDS: hess_lds_bytes.  A grid-stride loop over tiles, so any grid is correct.
template <typename T, int LT, bool NORM, int SP>
__global__ __launch_bounds__(kOrdThreads) void k_hess(HessParams P) {
  constexpr T kIS2 = T(kInvSqrt2d);
  constexpr int W = Vec16<T>::n;
  extern __shared__ __align__(16) unsigned char smem[];
  T* st = reinterpret_cast<T*>(smem);
  const int L = LT >= 0 ? LT : P.L;
  const int K = (L + 1) * (L + 1), R9 = 9 * K;
  const int pad = hess_pad<T>(L), S9 = R9 + pad;
  const int PT = LT >= 0 ? hess_points<T>(LT) : P.tile;
  const int tid = threadIdx.x, nt = blockDim.x;
  const OrdTable<T>& C = ord_table<T>(0);
  const int half = SP == 2 ? nt / 2 : nt;  // whole waves
  const int part = SP == 2 ? __builtin_amdgcn_readfirstlane(tid / half) : 0;
  const int it = tid - part * half;
  const int m = it / PT, p = it - m * PT;
  const bool lane_on = m <= L && !(part == 1 && m == 0);
  const int mm = m <= L ? m : L;
  const int lw = __builtin_amdgcn_readfirstlane(it / kWave * kWave / PT);
  const int l0 = lw <= L ? lw : L + 1;
  const int64_t tiles = (P.n + PT - 1) / PT;
  for (int64_t tile = xcd_slot(blockIdx.x, gridDim.x); tile < tiles; tile += gridDim.x) {
    const int64_t p0 = tile * PT;
    const int np = static_cast<int>(P.n - p0 < PT ? P.n - p0 : PT);
    const T* xp = static_cast<const T*>(P.xyz) + (p0 + (p < np ? p : np - 1)) * 3;
    const Point<T> pt = make_point<T, NORM>(xp[0], xp[1], xp[2]);
    T* gd = static_cast<T*>(P.d2Y) + p0 * R9;
    const int sh = ord_shift(gd);
    // the evaluation point and its powers in double, as in k_ord
    double ux = xp[0], uy = xp[1], uz = xp[2], ui = 1.0;
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
    // (x + i y)^(m-2) by squaring, then two more factors
    constexpr int kBits = LT < 0 ? 5 : (LT > 9 ? 4 : (LT > 5 ? 3 : (LT > 3 ? 2 : 1)));
    double c2 = 1.0, s2 = 0.0;
    {
      const int ex = mm >= 2 ? mm - 2 : 0;
      double bc = ux, bs = uy;
#pragma unroll
      for (int b = 0; b < kBits; ++b) {
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
    // the order's factor t, its gradient and its second derivatives xx and xy
    // (yy = -xx), for the columns +m (c_m) and -m (s_m)
    T tp = static_cast<T>(c0), tpx = static_cast<T>(fm * c1), tpy = static_cast<T>(-fm * s1);
    T tpA = static_cast<T>(fmm * c2), tpB = static_cast<T>(-fmm * s2);
    T tm = static_cast<T>(s0), tmx = static_cast<T>(fm * s1), tmy = static_cast<T>(fm * c1);
    T tmA = static_cast<T>(fmm * s2), tmB = static_cast<T>(fmm * c2);
    if (mm == 0) {  // one column: both signs write the same values
      tp = tm = kIS2;
      tpx = tpy = tmx = tmy = T(0);
    }
    if constexpr (SP == 2) {
      if (part == 1) {
        tp = tm;
        tpx = tmx;
        tpy = tmy;
        tpA = tmA;
        tpB = tmB;
      }
    }
    const T tp2x = tpx + tpx, tp2y = tpy + tpy, tm2x = tmx + tmx, tm2y = tmy + tmy;
    const T x = static_cast<T>(ux), y = static_cast<T>(uy), z = static_cast<T>(uz);
    const T x2 = x + x, y2 = y + y, z2 = z + z;
    const T ir2 = static_cast<T>(ui * ui);
    const T rho2 = static_cast<T>(ux * ux + uy * uy);
    HessChain<T> ch{z, rho2};
    T* base = st + sh + p * S9 + l0 * l0 + l0 + (SP == 2 && part == 1 ? -mm : mm);
    T* basm = base - 2 * mm;
    T fl = T(l0);
    // the columns of degree l (fl) at o and, with one wave per order, om
    auto entries = [&](T N, T* o, T* om, auto mul) {
      if constexpr (NORM) N *= ir2;
      const T q = N * ch.p, Tm = N * ch.e, Wn = N * ch.w;
      const T Nx = N * ch.x;
      const T Z = Nx * ch.p1, V = Nx * ch.e1, U = Nx * ((ch.x - T(1)) * ch.p2);
      const T Qx = mul(x, Tm), Qy = mul(y, Tm);
      const T xW = mul(x, Wn);
      const T Qxx = mul(x, xW) + Tm, Qxy = mul(y, xW), Qyy = mul(y, mul(y, Wn)) + Tm;
      const T Qxz = mul(x, V), Qyz = mul(y, V);
      const T hl = (T(0.5) * fl + T(1)) * q;  // (l + 2)/2 q
      auto col = [&](T* c, T t, T tx, T ty, T tx2, T ty2, T A, T B) {
        T hxx = mul(Qxx, t) + (mul(Qx, tx2) + mul(q, A));
        T hyy = mul(Qyy, t) + (mul(Qy, ty2) - mul(q, A));
        T hxy = mul(Qxy, t) + (mul(Qx, ty) + (mul(Qy, tx) + mul(q, B)));
        T hxz = mul(Qxz, t) + mul(Z, tx);
        T hyz = mul(Qyz, t) + mul(Z, ty);
        T hzz = mul(U, t);
        if constexpr (NORM) {
          // ls = l s, so that u enters as it is
          const T lt = fl * t, h = hl * lt;
          const T sx = Qx * lt + (q * (fl * tx) - h * x);
          const T sy = Qy * lt + (q * (fl * ty) - h * y);
          const T sz = Z * lt - h * z;
          const T ly = q * lt;
          hxx -= x2 * sx + ly;
          hyy -= y2 * sy + ly;
          hzz -= z2 * sz + ly;
          hxy -= x * sy + y * sx;
          hxz -= x * sz + z * sx;
          hyz -= y * sz + z * sy;
        }
        c[0] = hxx;
        c[K] = hxy;
        c[2 * K] = hxz;
        c[3 * K] = hxy;
        c[4 * K] = hyy;
        c[5 * K] = hyz;
        c[6 * K] = hxz;
        c[7 * K] = hyz;
        c[8 * K] = hzz;
      };
      col(o, tp, tpx, tpy, tp2x, tp2y, tpA, tpB);
      if constexpr (SP == 1) col(om, tm, tmx, tmy, tm2x, tm2y, tmA, tmB);
    };
    auto degree = [&](int l, T N, T inv) {
      if (lane_on && l >= mm) {
        entries(N, base, basm, MulPlain{});
        ch.advance(inv, MulPlain{});
      }
      fl += T(1);
      base += 2 * l + 2;
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
      for (int u = 0; u < kOrdStep; ++u) {
        if (l + u <= L) degree(l + u, Ac[2 * u], u + 1 < kOrdStep ? Ac[(2 * u + 3) % (2 * kOrdStep)] : Bc[1]);
        // one degree after the other: interleaved they take more registers
        asm volatile("" : "+v"(ch.p), "+v"(ch.p1), "+v"(ch.e), "+v"(ch.w));
      }
#pragma unroll
      for (int u = 0; u < 2 * kOrdStep; ++u) Ac[u] = Bc[u];
    }
    if constexpr (!NORM) {  // past reach2: once more, see HessChain
      if (lane_on && !(rho2 + z * z <= static_cast<T>(P.reach2))) {
        ch = HessChain<T>{z, rho2};
        T* o = st + sh + p * S9 + (SP == 2 && part == 1 ? -mm : mm);
        fl = T(mm);
#pragma unroll 1
        for (int l = mm; l <= L; ++l) {
          entries(C.a[l][2 * mm], o + l * l + l, o + l * l + l - 2 * mm, MulZero{});
          ch.advance(C.a[l + 1][2 * mm + 1], MulZero{});
          fl += T(1);
        }
      }
    }
    __syncthreads();
    const int cnt = np * R9;
    if (pad == 0) {
      ord_copy_out(st, sh, gd, cnt, tid, nt);
    } else if (sh == 0) {  // points of whole vectors, one between them; as ord_copy_out
      using V = typename Vec16<T>::type;
      const int rv = R9 / W, nv = np * rv;
      const __amdgpu_buffer_rsrc_t rs = stream_rsrc(gd, nv * 16);
      V* gv = reinterpret_cast<V*>(gd);
      const V* sv = reinterpret_cast<const V*>(st);
      constexpr int kLine = 128 / 16;
      int v0 = (kLine - static_cast<int>((reinterpret_cast<uintptr_t>(gv) / 16) % kLine)) % kLine;
      v0 = v0 < nv ? v0 : nv;
      const int v1 = v0 + (nv - v0) / kLine * kLine;
      for (int i0 = v0 + tid; i0 < v1; i0 += nt * kOrdBatch) {
        V v[kOrdBatch];
#pragma unroll
        for (int u = 0; u < kOrdBatch; ++u) {
          const int i = i0 + u * nt;
          if (i < v1) v[u] = sv[i + i / rv];
        }
#pragma unroll
        for (int u = 0; u < kOrdBatch; ++u)
          if (i0 + u * nt < v1) stream_store16(v[u], rs, (i0 + u * nt) * 16);
      }
      if (tid < v0) gv[tid] = sv[tid + tid / rv];
      if (tid < nv - v1) gv[v1 + tid] = sv[v1 + tid + (v1 + tid) / rv];
    } else {
      for (int i = tid; i < cnt; i += nt) gd[i] = st[sh + i + i / R9 * pad];
    }
    if (tile + gridDim.x < tiles) __syncthreads();
  }
}

}  // namespace sph
