// backward from the points, double
#include <utility>

#include "sph_vjp.inl"

namespace sph {
namespace {

using T = double;

template <bool NORM, int... Ls>
void fill(const void** out, std::integer_sequence<int, Ls...>) {
  const void* tbl[] = {reinterpret_cast<const void*>(&k_vjp<T, Ls, NORM, vjp_waves<T>(Ls)>)...};
  for (size_t i = 0; i < sizeof...(Ls); ++i) out[i] = tbl[i];
}

struct Tables {
  const void* fn[2][kCompileMax<T> + 1];
  Tables() {
    fill<false>(fn[0], std::make_integer_sequence<int, kCompileMax<T> + 1>{});
    fill<true>(fn[1], std::make_integer_sequence<int, kCompileMax<T> + 1>{});
  }
};

const Tables& tables() {
  static const Tables t;
  return t;
}

}  // namespace

KernelInfo vjp_info_f64(int L, int normalize) {
  if (L < 0 || L > kMaxLmax || (normalize != 0 && normalize != 1)) return KernelInfo{nullptr, 0, 0, 0, 0};
  if (L > kCompileMax<T>) return ord_info_f64(L, normalize, false, false, true);
  const int waves = vjp_waves<T>(L);
  const size_t lds = sizeof(T) * (static_cast<size_t>(kVjpPoints) * vjp_stride((L + 1) * (L + 1)) +
                                  static_cast<size_t>(3 * kWave) * (waves - 1));
  return KernelInfo{tables().fn[normalize][L], lds, lds, kVjpPoints, kWave * waves};
}

}  // namespace sph
