// backward from the points, float
#include <utility>

#include "sph_vjp.inl"

namespace sph {
namespace {

using T = float;

template <bool NORM, bool E3, int... Ls>
void fill(const void** out, std::integer_sequence<int, Ls...>) {
  const void* tbl[] = {reinterpret_cast<const void*>(&k_vjp<T, Ls, NORM, E3, vjp_waves<T>(Ls)>)...};
  for (size_t i = 0; i < sizeof...(Ls); ++i) out[i] = tbl[i];
}

struct Tables {
  const void* fn[2][2][kCompileMax<T> + 1];  // [normalize][e3nn]
  Tables() {
    using Ls = std::make_integer_sequence<int, kCompileMax<T> + 1>;
    fill<false, false>(fn[0][0], Ls{});
    fill<false, true>(fn[0][1], Ls{});
    fill<true, false>(fn[1][0], Ls{});
    fill<true, true>(fn[1][1], Ls{});
  }
};

const Tables& tables() {
  static const Tables t;
  return t;
}

}  // namespace

KernelInfo vjp_info_f32(int L, int normalize, int conv) {
  if (L < 0 || L > kMaxLmax || (normalize != 0 && normalize != 1)) return KernelInfo{nullptr, 0, 0, 0, 0};
  if (L > kCompileMax<T>) return ord_info_f32(L, normalize, false, false, true);
  const int waves = vjp_waves<T>(L);
  const size_t lds = sizeof(T) * (static_cast<size_t>(kVjpPoints) * vjp_stride((L + 1) * (L + 1)) +
                                  static_cast<size_t>(3 * kWave) * (waves - 1));
  return KernelInfo{tables().fn[normalize][conv > 0 ? 1 : 0][L], lds, lds, kVjpPoints, kWave * waves};
}

}  // namespace sph
