// Instantiations and lookup of k_expbwd for one element type SPH_T (suffix
// SPH_SUFFIX) and normalisation SPH_NORM.
#include <utility>

#include "sph_expbwd.inl"

#define SPH_CAT2(a, b) a##b
#define SPH_CAT(a, b) SPH_CAT2(a, b)

namespace sph {
namespace {

using T = SPH_T;
constexpr int kSlots = kExpandMaxL + 1;

template <int LT, int NPC, bool VEC, bool FEW>
const void* fn_ptr() {
  if constexpr (!expbwd_serves<T>(LT, NPC))
    return nullptr;
  else
    return reinterpret_cast<const void*>(&k_expbwd<T, LT, SPH_NORM != 0, NPC, expbwd_waves<T>(LT, NPC, VEC, FEW),
                                                 VEC && expbwd_vec<T>(LT, NPC)>);
}

template <int NPC, bool VEC, bool FEW, int... Ls>
void fill(const void** out, std::integer_sequence<int, Ls...>) {
  const void* tbl[] = {fn_ptr<Ls, NPC, VEC, FEW>()...};
  for (size_t i = 0; i < sizeof...(Ls); ++i) out[i] = tbl[i];
}

struct Tables {
  const void* fn[2][2][2][kSlots];  // [few environments][16 channels][whole vectors]
  Tables() {
    using Ls = std::make_integer_sequence<int, kSlots>;
    fill<8, false, false>(fn[0][0][0], Ls{});
    fill<8, true, false>(fn[0][0][1], Ls{});
    fill<16, false, false>(fn[0][1][0], Ls{});
    fill<16, true, false>(fn[0][1][1], Ls{});
    fill<8, false, true>(fn[1][0][0], Ls{});
    fill<8, true, true>(fn[1][0][1], Ls{});
    fill<16, false, true>(fn[1][1][0], Ls{});
    fill<16, true, true>(fn[1][1][1], Ls{});
  }
};

}  // namespace

const void* SPH_CAT(SPH_CAT(SPH_CAT(expbwd_fn_, SPH_SUFFIX), _n), SPH_NORM)(int L, int npc, bool vec, bool few) {
  static const Tables t;
  return L < 0 || L > kExpandMaxL ? nullptr : t.fn[few ? 1 : 0][npc == 16 ? 1 : 0][vec ? 1 : 0][L];
}

}  // namespace sph
