// double-backward kernels, double
#include <utility>

#include "sph_dbord.inl"
#include "sph_dbwd.inl"

namespace sph {
namespace {

using T = double;
constexpr int kSlots = kCompileMax<T> + 1;

struct Tables {
  const void* fn[2][kSlots];
  template <bool NORM, int... Ls>
  static void fill(const void** out, std::integer_sequence<int, Ls...>) {
    const void* tbl[] = {reinterpret_cast<const void*>(&k_dbwd<T, Ls, NORM, dbwd_waves<T>(Ls, NORM)>)...};
    for (int i = 0; i < kSlots; ++i) out[i] = tbl[i];
  }
  Tables() {
    fill<false>(fn[0], std::make_integer_sequence<int, kSlots>{});
    fill<true>(fn[1], std::make_integer_sequence<int, kSlots>{});
  }
};

}  // namespace

KernelInfo dbwd_info_f64(int L, int normalize) {
  if (L < 0 || L > kMaxLmax || (normalize != 0 && normalize != 1)) return KernelInfo{nullptr, 0, 0, 0, 0};
  if (L > kCompileMax<T>) {
    const void* fn = normalize ? reinterpret_cast<const void*>(&k_dbord<T, true>)
                               : reinterpret_cast<const void*>(&k_dbord<T, false>);
    const int points = dbord_points<T>(L);
    const size_t lds = dbord_lds_bytes<T>(L, points);
    return KernelInfo{fn, lds, lds, points, (points * (L + 1) + kWave - 1) / kWave * kWave};
  }
  static const Tables t;
  const int waves = dbwd_waves<T>(L, normalize == 1);
  const size_t lds = dbwd_lds_bytes<T>(L, waves);
  return KernelInfo{t.fn[normalize][L], lds, lds, kWave, kWave * waves};
}

}  // namespace sph
