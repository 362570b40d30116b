// Instantiations of the general score kernel (score.hip) that are picked at run time.
#include "launch.h"
#include "score.hip"

namespace palu {

namespace {

// waves8: four heads as 8 half-head wavefronts (two per SIMD) instead of 4 whole-head ones.
template <typename T, bool I4, int NKS>
ScoreFn score_fn_g(int lg, bool waves8) {
  if constexpr (NKS > 16) {
    return score_kernel<T, NKS, 2, 1, 4, I4>;
  } else {
    if (waves8) {
      if constexpr (NKS <= 8) { if (lg == 2) return score_kernel<T, NKS, 2, 4, 8, I4>; }
      if (lg == 1) return score_kernel<T, NKS, 2, 2, 8, I4>;
      return score_kernel<T, NKS, 2, 1, 8, I4>;
    }
    if constexpr (NKS <= 8) { if (lg == 2) return score_kernel<T, NKS, 4, 4, 4, I4>; }
    if (lg == 1) return score_kernel<T, NKS, 4, 2, 4, I4>;
    return score_kernel<T, NKS, 4, 1, 4, I4>;
  }
}
template <typename T, bool I4>
ScoreFn score_fn_t(int rc, int lg, bool w8) {
  switch (rc) {
    case 0: return score_fn_g<T, I4, 2>(lg, w8);
    case 1: return score_fn_g<T, I4, 4>(lg, w8);
    case 2: return score_fn_g<T, I4, 6>(lg, w8);
    case 3: return score_fn_g<T, I4, 8>(lg, w8);
    case 4: return score_fn_g<T, I4, 10>(lg, w8);
    case 5: return score_fn_g<T, I4, 12>(lg, w8);
    case 6: return score_fn_g<T, I4, 14>(lg, w8);
    case 7: return score_fn_g<T, I4, 16>(lg, w8);
    case 8: return score_fn_g<T, I4, 18>(lg, w8);
    case 9: return score_fn_g<T, I4, 20>(lg, w8);
    case 10: return score_fn_g<T, I4, 22>(lg, w8);
    case 11: return score_fn_g<T, I4, 24>(lg, w8);
    case 12: return score_fn_g<T, I4, 26>(lg, w8);
    case 13: return score_fn_g<T, I4, 28>(lg, w8);
    case 14: return score_fn_g<T, I4, 30>(lg, w8);
    default: return score_fn_g<T, I4, 32>(lg, w8);
  }
}
}  // namespace

ScoreFn score_fn(int act, bool i4, int cls_id, bool w8) {
  const int rc = cls_id / 3, lg = cls_id % 3;
  if (i4) return score_fn_t<F16, true>(rc, lg, w8);
  return act == PALU_F16 ? score_fn_t<F16, false>(rc, lg, w8) : score_fn_t<BF16, false>(rc, lg, w8);
}


}  // namespace palu
