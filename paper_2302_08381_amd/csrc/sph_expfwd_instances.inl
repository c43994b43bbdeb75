// Instantiations and lookup of k_expfwd for one element type SPH_T (suffix
// SPH_SUFFIX) and normalisation SPH_NORM.
#include <utility>

#include "sph_expfwd.inl"

#define SPH_CAT2(a, b) a##b
#define SPH_CAT(a, b) SPH_CAT2(a, b)

namespace sph {
namespace {

using T = SPH_T;
constexpr int kSlots = kCompileMax<T> + 1;
constexpr int kLayouts = 4;

// Layouts of the channels, groups of CW:  Three groups of four for 9..12
// channels where a part fits the block (float, l_max 6, 12 channels: 125 us
// against 190 as two groups of eight; l_max 8 195 and 244).
constexpr int layout_cw(int i) { return i == 0 || i == 2 ? 4 : 8; }
constexpr int layout_ng(int i) { return i == 2 ? 3 : (i == 3 ? 2 : 1); }
constexpr bool layout_serves(int L, int i) {
  return (L + 1) * (L + 2) / 2 * layout_ng(i) <= kWave * 4;
}
constexpr int layout_of(int L, int n_max) {
  return n_max <= 4 ? 0 : (n_max <= 8 ? 1 : (n_max <= 12 && layout_serves(L, 2) ? 2 : 3));
}

template <int LT, int I, int WV, bool VEC>
KernelInfo info() {
  constexpr int CW = layout_cw(I), NG = layout_ng(I);
  if constexpr (!layout_serves(LT, I) || (WV == 2 && expfwd_waves(LT, CW * NG, 1 << 20) != 2)) {
    return KernelInfo{nullptr, 0, 0, 0, 0};
  } else {
    return KernelInfo{reinterpret_cast<const void*>(&k_expfwd<T, LT, SPH_NORM != 0, CW, NG, WV, VEC>),
                      ExpFwd<T, LT, CW, NG, WV>::lds_bytes, 0, 0, kWave * WV};
  }
}

template <int I, int WV, bool VEC, int... Ls>
void fill_one(KernelInfo* out, std::integer_sequence<int, Ls...>) {
  const KernelInfo tbl[] = {info<Ls, I, WV, VEC>()...};
  for (size_t i = 0; i < sizeof...(Ls); ++i) out[i] = tbl[i];
}

struct Tables {
  KernelInfo k[kLayouts][2][2][kSlots];  // [layout][two waves][whole vectors]
  template <int I>
  void fill() {
    using Ls = std::make_integer_sequence<int, kSlots>;
    fill_one<I, 4, false>(k[I][0][0], Ls{});
    fill_one<I, 4, true>(k[I][0][1], Ls{});
    fill_one<I, 2, false>(k[I][1][0], Ls{});
    fill_one<I, 2, true>(k[I][1][1], Ls{});
  }
  Tables() {
    fill<0>();
    fill<1>();
    fill<2>();
    fill<3>();
  }
};

}  // namespace

KernelInfo SPH_CAT(SPH_CAT(SPH_CAT(expfwd_info_, SPH_SUFFIX), _n), SPH_NORM)(int L, int n_max, bool aligned, int64_t n_env) {
  static const Tables t;
  const int i = layout_of(L, n_max);
  const bool vec = aligned && n_max == layout_cw(i) * layout_ng(i);
  return t.k[i][expfwd_waves(L, n_max, n_env) == 2 ? 1 : 0][vec ? 1 : 0][L];
}

}  // namespace sph
