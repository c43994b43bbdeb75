// radial expansion kernels, double
#include <utility>

#include "sph_expand.inl"

namespace sph {
namespace {

using T = double;

// l_max <= 8: compile-time degrees; larger: the run-time-degree kernel of
// the m-extent bucket.
constexpr int kSpecMax = 8;

// The run-time degrees, for the buckets that reach past the compile-time ones.
template <bool NORM, int ACC, int MM>
const void* bucket_ptr() {
  if constexpr (MM > kSpecMax)
    return reinterpret_cast<const void*>(&k_expand<T, MM, -1, NORM, ACC>);
  else
    return nullptr;
}

template <bool NORM, int ACC, int... Is>
void fill_expand(const void** out, std::integer_sequence<int, Is...>) {
  const void* tbl[] = {bucket_ptr<NORM, ACC, kBuckets[Is]>()...};
  for (size_t i = 0; i < sizeof...(Is); ++i) out[i] = tbl[i];
}

// The compile-time degrees serve more than 16 channels here.
template <bool NORM, int ACC, int LT>
const void* spec_ptr() {
  if constexpr (ACC == 8 || expand_acc(LT, kExpFwdChannels + 1) == 4)
    return reinterpret_cast<const void*>(&k_expand<T, LT, LT, NORM, ACC>);
  else
    return nullptr;
}

template <bool NORM, int ACC, int... Ls>
void fill_spec(const void** out, std::integer_sequence<int, Ls...>) {
  const void* tbl[] = {spec_ptr<NORM, ACC, Ls>()...};
  for (size_t i = 0; i < sizeof...(Ls); ++i) out[i] = tbl[i];
}

// The run-time-degree backward, for the buckets that reach past the
// compile-time one.
template <bool NORM, int NPC, int MM>
const void* bwd_ptr() {
  if constexpr (!expbwd_serves<T>(MM, NPC))
    return reinterpret_cast<const void*>(&k_expand_bwd<T, MM, NORM, NPC>);
  else
    return nullptr;
}

template <bool NORM, int NPC, int... Is>
void fill_bwd(const void** out, std::integer_sequence<int, Is...>) {
  const void* tbl[] = {bwd_ptr<NORM, NPC, kBuckets[Is]>()...};
  for (size_t i = 0; i < sizeof...(Is); ++i) out[i] = tbl[i];
}

struct Tables {
  const void* fn[2][2][kNumBuckets];  // [normalize][ACC == 8]
  const void* spec[2][2][kSpecMax + 1];
  const void* bwd[2][2][kNumBuckets];  // [normalize][NPC == 16]
  Tables() {
    using Is = std::make_integer_sequence<int, kNumBuckets>;
    fill_bwd<false, 8>(bwd[0][0], Is{});
    fill_bwd<true, 8>(bwd[1][0], Is{});
    fill_bwd<false, 16>(bwd[0][1], Is{});
    fill_bwd<true, 16>(bwd[1][1], Is{});
    fill_expand<false, 4>(fn[0][0], std::make_integer_sequence<int, kNumBuckets>{});
    fill_expand<true, 4>(fn[1][0], std::make_integer_sequence<int, kNumBuckets>{});
    fill_expand<false, 8>(fn[0][1], std::make_integer_sequence<int, kNumBuckets>{});
    fill_expand<true, 8>(fn[1][1], std::make_integer_sequence<int, kNumBuckets>{});
    fill_spec<false, 4>(spec[0][0], std::make_integer_sequence<int, kSpecMax + 1>{});
    fill_spec<true, 4>(spec[1][0], std::make_integer_sequence<int, kSpecMax + 1>{});
    fill_spec<false, 8>(spec[0][1], std::make_integer_sequence<int, kSpecMax + 1>{});
    fill_spec<true, 8>(spec[1][1], std::make_integer_sequence<int, kSpecMax + 1>{});
  }
};

const Tables& tables() {
  static const Tables t;
  return t;
}

}  // namespace

KernelInfo expand_info_f64(int L, int normalize, int n_max, bool aligned, bool two) {
  if (L < 0 || L > kMaxLmax || (normalize != 0 && normalize != 1) || n_max < 1) return KernelInfo{nullptr, 0, 0, 0, 0};
  if (expfwd_serves(L, n_max))
    return normalize ? expfwd_info_f64_n1(L, n_max, aligned, two) : expfwd_info_f64_n0(L, n_max, aligned, two);
  const Tables& t = tables();
  const int a = expand_acc(L, n_max) == 8 ? 1 : 0;
  const void* fn = L <= kSpecMax ? t.spec[normalize][a][L] : t.fn[normalize][a][bucket_index(L)];
  return KernelInfo{fn, 0, 0, 0, kExpandThreads};
}

KernelInfo expand_bwd_info_f64(int L, int normalize, int n_max, bool aligned, int64_t n, int64_t n_env, int cus) {
  if (L < 0 || L > kMaxLmax || (normalize != 0 && normalize != 1) || n_max < 1 || n_max > 16)
    return KernelInfo{nullptr, 0, 0, 0, 0};
  const int npc = n_max > 8 ? 16 : 8;
  if (expbwd_serves<T>(L, npc)) {
    const bool vec = n_max == npc && aligned;
    const bool few = n_env <= 2 * cus;
    const void* fn = normalize ? expbwd_fn_f64_n1(L, npc, vec, few) : expbwd_fn_f64_n0(L, npc, vec, few);
    const int waves = expbwd_waves<T>(L, npc, vec, few);
    const int slices = expbwd_slices<T>(npc, n, n_env);
    KernelInfo ki{fn, expbwd_lds_bytes<T>(L, npc, slices, waves), 0, 1, kWave * waves};
    ki.slices = slices;
    return ki;
  }
  // one G slice where two would not fit (chunks then stop at every
  // environment's end)
  const int slices = expand_bwd_lds_bytes<T>(L, npc, 2) <= 160 * 1024 ? 2 : 1;
  KernelInfo ki{tables().bwd[normalize][npc == 16 ? 1 : 0][bucket_index(L)], expand_bwd_lds_bytes<T>(L, npc, slices), 0, 1,
                kWave};
  ki.slices = slices;
  return ki;
}

}  // namespace sph
