// explicit Hessian kernels, float
#include <utility>

#include "sph_hess.inl"

namespace sph {
namespace {

using T = float;
constexpr int kSlots = kCompileMax<T> + 1;

struct Tables {
  const void* fn[2][kSlots + 1];  // last: the run-time degree
  template <bool NORM, int... Ls>
  static void fill(const void** out, std::integer_sequence<int, Ls...>) {
    const void* tbl[] = {reinterpret_cast<const void*>(&k_hess<T, Ls, NORM, hess_split(Ls)>)...,
                         reinterpret_cast<const void*>(&k_hess<T, -1, NORM, hess_split(kSlots)>)};
    for (int i = 0; i <= kSlots; ++i) out[i] = tbl[i];
  }
  Tables() {
    fill<false>(fn[0], std::make_integer_sequence<int, kSlots>{});
    fill<true>(fn[1], std::make_integer_sequence<int, kSlots>{});
  }
};

}  // namespace

KernelInfo hess_info_f32(int L, int normalize) {
  if (L < 0 || L > kMaxLmax || (normalize != 0 && normalize != 1)) return KernelInfo{nullptr, 0, 0, 0, 0};
  static const Tables t;
  const int points = hess_points<T>(L);
  const size_t lds = hess_lds_bytes<T>(L, points);
  return KernelInfo{t.fn[normalize][L < kSlots ? L : kSlots], lds, lds, points,
                    hess_split(L) * ((points * (L + 1) + kWave - 1) / kWave * kWave)};
}

}  // namespace sph
