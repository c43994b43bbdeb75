// Internal interface between the C ABI (sph_api.cpp) and the kernel
// translation units.  Not installed; the public interface is include/sph.h.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace sph {

// Largest supported l_max (the m-extent of the widest kernel bucket).
constexpr int kMaxLmax = 32;

// Kernel parameters of the forward / batched kernel (one struct argument so
// the same layout serves direct launches and graph kernel nodes).
struct FwdParams {
  const void* xyz;        // [n,3]
  int64_t n;              // points
  int32_t L;              // l_max (runtime-degree kernels)
  void* Y;                // [n,K]
  void* dY;               // [n,3,K] or null
  const void* gY;         // [n,K] or null (fused backward)
  void* gxyz;             // [n,3] (required iff gY)
  const int64_t* offsets; // CSR offsets or null (no validation)
  int64_t n_env;
  int32_t* status;        // device status word or null
  int32_t tile = 0;       // points per tile (k_ord)
  int32_t conv = 0;       // 0: this library's harmonics; 1 + normalization: e3nn's factors, and grad_xyz along
                          // the axes of the points before their permutation (k_fwd, k_vjp, k_ord)
};

// Largest l_max of the compile-time forward kernels; k_ord serves the rest.
template <typename T>
inline constexpr int kCompileMax = sizeof(T) == 4 ? 12 : 8;

struct BwdParams {
  const void* dY;
  const void* gY;
  int64_t n;
  int32_t K;
  void* gxyz;
};

struct DbwdParams {
  const void* xyz;
  const void* gY;
  const void* v;
  int64_t n;
  int32_t L;
  void* ggY;   // nullable
  void* gxyz2; // nullable
  int32_t tile;  // points per block
  double reach2; // see scaled_reach2 (k_dbord)
};

// Explicit Hessians (k_hess).
struct HessParams {
  const void* xyz;  // [n,3]
  int64_t n;
  int32_t L;
  void* d2Y;        // [n,3,3,K]
  int32_t tile;     // points per block
  double reach2;    // see scaled_reach2
};

// Squared distance from the origin up to which the scaled harmonics of
// l_max, their derivatives and every product on the way to them are within
// the type's range (r^l times the largest of their factors, below 1e10 for
// every l <= 32).
inline double scaled_reach2(int L, bool f64) {
  return std::pow(f64 ? 1e298 : 1e28, 2.0 / (L > 2 ? L : 2));
}

// Radial expansion over CSR environments (k_expand).
struct ExpandParams {
  const void* xyz;         // [n,3]
  const void* R;           // [n, L+1, n_max]
  const int64_t* offsets;  // [n_env+1]
  int64_t n_env;
  int64_t n;               // points (offsets[n_env] when consistent)
  int32_t L;
  int32_t n_max;
  int32_t chunk;           // points per LDS chunk (<= 128)
  void* c;                 // [n_env, n_max, K]
  int32_t* status;         // device status word or null
};

// LDS layout of one block (elements of T):
//   Y tile:   chunk rows of stride expand_ystride(K) (odd: conflict-free
//             column reads and row writes)
//   R tile:   chunk rows of (L+1) * NP, NP = n_max rounded up to the
//             accumulator width (4 or 8), zero padded, so each thread's
//             channels are aligned 16-byte vectors
//   C tile:   NP * K partial sums
__host__ __device__ constexpr int expand_ystride(int K) { return K | 1; }
__host__ __device__ constexpr int expand_np(int n_max, int acc) { return (n_max + acc - 1) / acc * acc; }
// Channels per accumulator item: 8 where 4 would need more than one pass of
// the block's 128 threads over the (column, channel group) items and there
// are more than 4 channels; else 4.  (Measured on 20 000 environments with 8
// channels: 8 is faster at l_max 8 and 12, 4 at l_max 3 and 6.)
__host__ __device__ constexpr int expand_acc(int L, int n_max) {
  return n_max > 4 && (L + 1) * (L + 1) * expand_np(n_max, 4) / 4 > 128 ? 8 : 4;
}
template <typename T>
__host__ __device__ constexpr size_t expand_lds_bytes(int L, int n_max, int chunk) {
  const int K = (L + 1) * (L + 1);
  // the Y tile is rounded to 16 bytes so the R tile starts aligned
  const size_t ytile = (static_cast<size_t>(chunk) * expand_ystride(K) * sizeof(T) + 15) & ~size_t(15);
  const int np = expand_np(n_max, expand_acc(L, n_max));
  return ytile + sizeof(T) * (static_cast<size_t>(chunk) * (L + 1) * np + static_cast<size_t>(np) * K);
}

// Where the compile-time kernel (k_expfwd) serves: up to l_max 12 and 16
// channels (24 channels, float l_max 8, 5000 environments: 131 us in k_expand
// against 145 as two groups of 16).  Double past l_max 8, 3000 environments,
// against run-time degrees: l_max 9 3 channels 80 -> 36 us, 12 194 -> 78;
// l_max 10 8 channels 134 -> 65, 16 193 -> 157.
constexpr int kExpandMaxL = 12;
constexpr int kExpFwdChannels = 16;
constexpr bool expfwd_serves(int L, int n_max) { return L <= kExpandMaxL && n_max <= kExpFwdChannels; }
// Up to l_max 4 and 8 channels it exists on two waves as well as four, see
// expfwd_two_waves for the choice (12 channels, float l_max 4, 20 000
// environments: 83 us on two, 80 on four).
constexpr bool expfwd_on_two(int L, int n_max) { return L <= 4 && n_max <= 8; }
// Two waves, whose blocks are more numerous, where there are more environments
// than four-wave blocks are resident (two / four waves, 8 channels, 20 000
// environments of 68 points: float l_max 4 57 / 67 us, double l_max 4 117 /
// 166; 2000 of 68, float l_max 3 8.1 / 13.4), and where the environments are
// short and fill the CUs twice (1000 of 16, double l_max 4 7.4 / 10.5).
// Long environments that are resident at once are four waves' (700 of 600,
// float l_max 3 21.4 / 19.3, 5 channels 27.8 / 23.1).
constexpr bool expfwd_two_waves(int64_t n, int64_t n_env, int64_t resident4, int cus) {
  return n_env > resident4 || (n_env > 2 * cus && n < 128 * n_env);
}

// Backward of the radial expansion (k_expand_bwd).
struct ExpandBwdParams {
  const void* xyz;         // [n,3]
  const void* R;           // [n, L+1, n_max]
  const int64_t* offsets;  // [n_env+1]
  int64_t n_env;
  int64_t n;
  int32_t L;
  int32_t n_max;
  const void* gc;          // [n_env, n_max, K] upstream gradient of c
  void* gxyz;              // [n,3] or null
  void* gR;                // [n, L+1, n_max] or null
  int32_t* status;         // device status word or null
  int32_t slices;          // G slices: environments a chunk may run through
};
// Row stride (elements) of the backward's LDS radial tile: (L+1) * np
// channels, padded so that a row spans an odd number of 16-byte vectors
// (lanes reading their rows as 16-byte vectors hit distinct banks).
template <typename T>
__host__ __device__ constexpr int expand_bwd_row_stride(int L, int np) {
  constexpr int W = 16 / static_cast<int>(sizeof(T));
  const int s = (L + 1) * np;
  return (s / W) % 2 == 1 ? s : s + W;
}
// LDS of one block of the run-time-degree backward: `slices` environment
// gradients G as [K][np] (two where a chunk may span two environments).
template <typename T>
__host__ __device__ constexpr size_t expand_bwd_lds_bytes(int L, int np, int slices) {
  return sizeof(T) * static_cast<size_t>(slices) * (L + 1) * (L + 1) * np;
}

// The compile-time backward (k_expbwd): environments a chunk may run through,
// and its LDS: the radial tile of 64 points, `slices` G slices and the sums of
// the waves past the first.
constexpr int kExpBwdSlices = 4;
// Waves that share a tile's degrees.  Twice the waves of a CU on the same LDS,
// against order-m tables formed twice.  Float, 20 000 environments, 1 / 2 / 4
// waves: 8 channels l_max 3 72 / 73 us, l_max 4 88.7 / 88.6, l_max 8 - / 210 /
// 240, l_max 12 - / 455 / 339; 16 channels (10 000) l_max 12 - / 832 / 508.
// Double, 8 channels l_max 3 180 / 201, l_max 8 - / 490 / 612; 3000 environments
// l_max 10 - / 116 / 160.
// Where it says one, two all the same
//   for the general copies (vec: whole-vector rows) of the largest of those
//   degrees (float 5 channels l_max 4, 5000 environments of 200 points 113 us
//   on one, 82 on two; double l_max 5 30 % fewer);
//   and in double, whose registers leave a SIMD one wave, for few environments
//   (at most two a CU): 60 of 3000 points, 8 channels l_max 5 411 us on one,
//   270 on two; 12 channels l_max 3 441 and 272, but 700 of 300 56 and 67.
template <typename T>
constexpr int expbwd_waves(int L, int npc, bool vec, bool few) {
  if (L <= (npc == 8 ? (sizeof(T) == 4 ? 4 : 5) : 3)) {
    if (npc == 8 && L >= 4 && !vec) return 2;
    if (sizeof(T) == 8 && few && (npc == 16 || L == 5)) return 2;
    return 1;
  }
  return L >= (npc == 8 && sizeof(T) == 4 ? 12 : 11) ? 4 : 2;
}
// Environments per chunk: four with 8 channels (l_max 8 float 210 us against
// 221 with two, double 490 and 533; all eight that a wider walk would allow
// cost 2-3 % there), two with 16, whose slices would cost blocks (float
// l_max 6 367 us against 415 with four), unless the environments have under 12
// points on average and two would leave most lanes idle (16 channels, l_max 6,
// 100 000 environments of 6 points: float 367 us with four, 479 with two;
// double 676 with three, 886 with two).
template <typename T>
constexpr int expbwd_slices(int npc, int64_t n, int64_t n_env) {
  if (npc == 8) return kExpBwdSlices;
  return n / (n_env > 0 ? n_env : 1) >= 12 ? 2 : (sizeof(T) == 4 ? 4 : 3);
}
// Where the compile-time kernel is the faster one: up to l_max 12, but not
// double with 9..16 channels past l_max 6, whose registers spill (10 000
// environments, l_max 8: 716 us against the run-time-degree kernel's 539;
// l_max 6 356 against 400).  Double past l_max 8, 3000 environments, 8
// channels: l_max 9 99 us against 164, l_max 12 156 against 255.
template <typename T>
constexpr bool expbwd_serves(int L, int npc) {
  return L <= kExpandMaxL && !(sizeof(T) == 8 && npc == 16 && L >= 7);
}
template <typename T>
constexpr size_t expbwd_lds_bytes(int L, int np, int slices, int waves) {
  return sizeof(T) * (static_cast<size_t>(64) * expand_bwd_row_stride<T>(L, np) +
                      static_cast<size_t>(slices) * (L + 1) * (L + 1) * np + static_cast<size_t>(3 * 64) * (waves - 1));
}

// A kernel's host stub, its dynamic LDS bytes (for the l_max it was looked
// up with), and for the forward with derivatives the LDS bytes when the
// backward is fused (the extra upstream-gradient tile); tile_points is the
// number of points one block covers per tile and block its threads.
struct KernelInfo {
  const void* fn;
  size_t lds_bytes;
  size_t lds_bytes_bwd;
  int tile_points;
  int block;
  int blocks_per_cu = 0;  // plain calls: 1: a resident grid (occupancy x CUs) loops over tiles; 0: one tile per block
  int slices = 0;         // the expansion backward: G slices per block
};

// Per element type (suffix f32 / f64) and normalisation; fn == nullptr when
// the arguments are out of range or the variant does not exist for l_max.
//   values:      Y only (one lane per point, 64-point tiles, 64 threads)
//   derivatives: four lanes per point, 32- or 16-point tiles (one lane per point
//                and 64-point tiles for the one-lane kernel); mode
//                kDerivStore (Y and dY), kDerivFusedStore (Y, dY and the
//                fused backward), kDerivFused (Y and the fused backward)
// Variants (the batched autotuner's candidates; two may name one kernel):
//   kVarDefault  the one-lane kernel for l_max <= 1; else the compile-time
//                (unrolled) kernel where one exists, on its
//                default tile (32 points on two waves for float l_max <= 8,
//                the degree-split tile where that measured faster, else 16
//                points on one wave); past them k_ord (not in these tables,
//                see ord_info)
//   kVarTile16   the compile-time kernel on an unsplit 16-point, one-wave tile
//   kVarRuntime  the unsplit run-time-degree (not unrolled) kernel
//   kVarSplit    a degree-split kernel: the compile-time one (float l_max
//                9..12, double 4..8) or the run-time-degree one (larger
//                l_max, no fused backward)
//   kVarLane     l_max <= 3: one lane per point, 64-point one-wave tiles
enum DerivMode { kDerivStore = 0, kDerivFusedStore = 1, kDerivFused = 2, kNumDerivModes = 3 };
enum FwdVariant { kVarDefault = 0, kVarTile16 = 1, kVarRuntime = 2, kVarSplit = 3, kVarLane = 4, kNumFwdVariants = 5 };
KernelInfo fwd_values_f32_n0(int L, int variant);
KernelInfo fwd_values_f32_n1(int L, int variant);
KernelInfo fwd_values_f64_n0(int L, int variant);
KernelInfo fwd_values_f64_n1(int L, int variant);
KernelInfo fwd_derivs_f32_n0_m0(int L, int variant);
KernelInfo fwd_derivs_f32_n0_m1(int L, int variant);
KernelInfo fwd_derivs_f32_n0_m2(int L, int variant);
KernelInfo fwd_derivs_f32_n1_m0(int L, int variant);
KernelInfo fwd_derivs_f32_n1_m1(int L, int variant);
KernelInfo fwd_derivs_f32_n1_m2(int L, int variant);
KernelInfo fwd_derivs_f64_n0_m0(int L, int variant);
KernelInfo fwd_derivs_f64_n0_m1(int L, int variant);
KernelInfo fwd_derivs_f64_n0_m2(int L, int variant);
KernelInfo fwd_derivs_f64_n1_m0(int L, int variant);
KernelInfo fwd_derivs_f64_n1_m1(int L, int variant);
KernelInfo fwd_derivs_f64_n1_m2(int L, int variant);
// l_max past the compile-time kernels (kCompileMax): k_ord for the outputs
// asked for, tile_points points per block (the launch sets FwdParams::tile).
KernelInfo ord_info_f32(int L, int normalize, bool store_y, bool store_dy, bool bwd);
KernelInfo ord_info_f64(int L, int normalize, bool store_y, bool store_dy, bool bwd);
// Backward from the points: the compile-time kernel of L, or k_ord past them.
KernelInfo vjp_info_f32(int L, int normalize, int conv);
KernelInfo vjp_info_f64(int L, int normalize, int conv);
KernelInfo bwd_info_f32(int L);
KernelInfo bwd_info_f64(int L);
KernelInfo dbwd_info_f32(int L, int normalize);
KernelInfo dbwd_info_f64(int L, int normalize);
// Explicit Hessians: k_hess with L at compile time up to kCompileMax, else the
// run-time one; tile_points points per block.
KernelInfo hess_info_f32(int L, int normalize);
KernelInfo hess_info_f64(int L, int normalize);
// Radial expansion: k_expfwd where it serves (lds_bytes set; aligned: R starts
// on a 16-byte boundary); else k_expand, compile-time degrees for float
// L <= 12 and double L <= 8, the m-extent bucket of L past them, with the
// accumulator width expand_acc(L, n_max), block = 128 threads and lds_bytes
// left 0 (they depend on n_max and the chunk, see expand_lds_bytes).
// two: on two waves (expfwd_on_two).
KernelInfo expand_info_f32(int L, int normalize, int n_max, bool aligned, bool two);
KernelInfo expand_info_f64(int L, int normalize, int n_max, bool aligned, bool two);
KernelInfo expfwd_info_f32_n0(int L, int n_max, bool aligned, bool two);
KernelInfo expfwd_info_f32_n1(int L, int n_max, bool aligned, bool two);
KernelInfo expfwd_info_f64_n0(int L, int n_max, bool aligned, bool two);
KernelInfo expfwd_info_f64_n1(int L, int n_max, bool aligned, bool two);
// Its backward: channels padded to 8 or 16 (n_max <= 16); aligned: R and
// grad_R start on 16-byte boundaries; cus: the device's; slices: the G slices
// of a block.
KernelInfo expand_bwd_info_f32(int L, int normalize, int n_max, bool aligned, int64_t n, int64_t n_env, int cus);
KernelInfo expand_bwd_info_f64(int L, int normalize, int n_max, bool aligned, int64_t n, int64_t n_env, int cus);
// The compile-time backward (L <= kExpandMaxL): the padded channel count npc
// (8 or 16), with or without the whole-vector copies, on the waves of
// expbwd_waves.
const void* expbwd_fn_f32_n0(int L, int npc, bool vec, bool few);
const void* expbwd_fn_f32_n1(int L, int npc, bool vec, bool few);
const void* expbwd_fn_f64_n0(int L, int npc, bool vec, bool few);
const void* expbwd_fn_f64_n1(int L, int npc, bool vec, bool few);
// e3nn's conventions: the permuted coordinates and the in-place conversion
// of Y and dY (dtype64: double, else float).
hipError_t e3nn_coordinates_launch(int dtype64, const void* xyz, int64_t n, void* out, hipStream_t s);
hipError_t e3nn_convert_launch(int dtype64, int64_t n, int L, int normalization, void* Y, void* dY,
                               hipStream_t s);

}  // namespace sph
