// Instantiations of the whole-head score kernel (score16.hip), one query per head, and of its 8-bit variant.
#include "launch.h"
#include "score16.hip"
#include "score8.hip"

#ifndef PALU_SCORE_FLAT
#define PALU_SCORE_FLAT 0
#endif

namespace palu {

namespace {
constexpr bool kFlat = PALU_SCORE_FLAT != 0;

// unquantized latents, ranks 64 .. 256, one query per head: one whole head per wavefront (score16.hip); 1, 2 or 4 groups of at
// most 256 columns in all
template <typename T, int NK>
ScoreFn score16_fn_g(int lg) {
  if constexpr (NK <= 2) { if (lg == 2) return score16_kernel<T, NK, 4, 1, 0, kFlat>; }
  if constexpr (NK <= 4) { if (lg == 1) return score16_kernel<T, NK, 2, 1, 0, kFlat>; }
  return lg == 0 ? score16_kernel<T, NK, 1, 1, 0, kFlat> : nullptr;
}
template <typename T>
ScoreFn score16_fn_t(int rc, int lg) {
  switch (rc) {
    case 1: return score16_fn_g<T, 2>(lg);
    case 2: return score16_fn_g<T, 3>(lg);
    case 3: return score16_fn_g<T, 4>(lg);
    case 4: return score16_fn_g<T, 5>(lg);
    case 5: return score16_fn_g<T, 6>(lg);
    case 6: return score16_fn_g<T, 7>(lg);
    default: return score16_fn_g<T, 8>(lg);
  }
}
}  // namespace

template <>
ScoreFn score16_fn<kFlat>(int act, int rc, int lg) {
  return act == PALU_F16 ? score16_fn_t<F16>(rc, lg) : score16_fn_t<BF16>(rc, lg);
}

template <>
ScoreFn score16_mixed_fn<kFlat>(int act) { return act == PALU_F16 ? score16_mixed_kernel<F16, kFlat> : score16_mixed_kernel<BF16, kFlat>; }

#if !PALU_SCORE_FLAT
namespace {
template <int NK>
ScoreFn score8_fn_g(int lg) {
  if constexpr (NK <= 2) { if (lg == 2) return score8_kernel<NK, 4>; }
  if constexpr (NK <= 4) { if (lg == 1) return score8_kernel<NK, 2>; }
  return lg == 0 ? score8_kernel<NK, 1> : nullptr;
}
}  // namespace

ScoreFn score8_fn(int rc, int lg) {
  switch (rc) {
    case 1: return score8_fn_g<2>(lg);
    case 2: return score8_fn_g<3>(lg);
    case 3: return score8_fn_g<4>(lg);
    case 4: return score8_fn_g<5>(lg);
    case 5: return score8_fn_g<6>(lg);
    case 6: return score8_fn_g<7>(lg);
    default: return score8_fn_g<8>(lg);
  }
}

int launch_fold8(const Fold8Args& a, hipStream_t s) {
  hipLaunchKernelGGL(fold8_kernel<F16>, dim3((unsigned)a.meta.n_heads, 4u), dim3(256), 0, s, a);
  return hipGetLastError() == hipSuccess ? PALU_OK : PALU_ERR_HIP;
}
#endif

}  // namespace palu
