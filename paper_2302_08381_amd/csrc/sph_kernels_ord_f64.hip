// one lane per (point, order): degrees past the compile-time kernels, double
#include "sph_ord.inl"

namespace sph {
namespace {

using T = double;

template <bool NORM, bool SPLIT>
const void* pick(bool store_y, bool store_dy, bool bwd) {
  if (store_dy)
    return bwd ? reinterpret_cast<const void*>(&k_ord<T, NORM, true, true, true, SPLIT>)
               : reinterpret_cast<const void*>(&k_ord<T, NORM, true, true, false, SPLIT>);
  if constexpr (SPLIT) {
    return nullptr;
  } else {
    if (bwd)
      return store_y ? reinterpret_cast<const void*>(&k_ord<T, NORM, true, false, true, false>)
                     : reinterpret_cast<const void*>(&k_ord<T, NORM, false, false, true, false>);
    return reinterpret_cast<const void*>(&k_ord<T, NORM, true, false, false, false>);
  }
}

}  // namespace

KernelInfo ord_info_f64(int L, int normalize, bool store_y, bool store_dy, bool bwd) {
  if (L <= kCompileMax<T> || L > kMaxLmax || (normalize != 0 && normalize != 1)) return KernelInfo{nullptr, 0, 0, 0, 0};
  const OrdShape sh = ord_shape<T>(L, store_y, store_dy, bwd);
  const void* fn = normalize ? (sh.split ? pick<true, true>(store_y, store_dy, bwd) : pick<true, false>(store_y, store_dy, bwd))
                             : (sh.split ? pick<false, true>(store_y, store_dy, bwd) : pick<false, false>(store_y, store_dy, bwd));
  const int waves = ((L + 1) * sh.points + kWave - 1) / kWave * (sh.split ? 2 : 1);
  const size_t lds = ord_lds_bytes<T>(L, sh.points, store_y, store_dy, bwd);
  return KernelInfo{fn, lds, lds, sh.points, waves * kWave};
}

}  // namespace sph
