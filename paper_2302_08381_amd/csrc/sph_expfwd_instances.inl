// Instantiations and lookup of k_expfwd for one element type SPH_T (suffix
// SPH_SUFFIX) and normalisation SPH_NORM.
#include <utility>

#include "sph_expfwd.inl"

#define SPH_CAT2(a, b) a##b
#define SPH_CAT(a, b) SPH_CAT2(a, b)

namespace sph {
namespace {

using T = SPH_T;
constexpr int kSlots = kExpandMaxL + 1;
constexpr int kLayouts = 6;

// Layouts of the channels, groups of CW: 4, 8, three of 4, two of 8, and in
// double 6 and two of 6.  Three groups of four for 9..12 channels where a part
// fits the block (float, 12 channels, 20 000 environments: l_max 6 125 us
// against 190 as two groups of eight; l_max 8 195 and 244).  In double the LDS
// tile of the padded channels costs blocks: six for 5 and 6 channels up to
// l_max 7 (5 channels, 10 000 environments, against eight: l_max 4 51 and 66
// us, l_max 5 65 and 86, l_max 6 85 and 92, l_max 7 92 and 133; but l_max 8
// 171 and 147; float l_max 8, 20 000, 128 and 131), two of six for 9..12 at
// l_max 8 (9 channels 181 against 213 as three of four; l_max 6 149 and 134).
constexpr int layout_cw(int i) { return i == 0 || i == 2 ? 4 : (i >= 4 ? 6 : 8); }
constexpr int layout_ng(int i) { return i == 2 ? 3 : (i == 3 || i == 5 ? 2 : 1); }
constexpr bool layout_serves(int L, int i) {
  if (i == 4) return sizeof(T) == 8 && L <= 7;
  if (i == 5) return sizeof(T) == 8 && L >= 8 && (L + 1) * (L + 2) <= kWave * 4;
  return (L + 1) * (L + 2) / 2 * layout_ng(i) <= kWave * 4;
}
constexpr int layout_of(int L, int n_max) {
  if (n_max <= 4) return 0;
  if (n_max <= 6 && layout_serves(L, 4)) return 4;
  if (n_max <= 8) return 1;
  if (n_max > 12) return 3;
  return layout_serves(L, 5) ? 5 : (layout_serves(L, 2) ? 2 : 3);
}

template <int LT, int I, int WV, bool VEC>
KernelInfo info() {
  constexpr int CW = layout_cw(I), NG = layout_ng(I);
  if constexpr (!layout_serves(LT, I) || (WV == 2 && !expfwd_on_two(LT, CW * NG))) {
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
    fill<4>();
    fill<5>();
  }
};

}  // namespace

KernelInfo SPH_CAT(SPH_CAT(SPH_CAT(expfwd_info_, SPH_SUFFIX), _n), SPH_NORM)(int L, int n_max, bool aligned, bool two) {
  static const Tables t;
  const int i = layout_of(L, n_max);
  const bool vec = aligned && n_max == layout_cw(i) * layout_ng(i);
  return t.k[i][two && expfwd_on_two(L, n_max) ? 1 : 0][vec ? 1 : 0][L];
}

}  // namespace sph
