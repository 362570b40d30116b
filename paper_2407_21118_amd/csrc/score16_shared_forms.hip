// Instantiations of the whole-head score kernel (score16.hip) for several queries per key/value head, and for 4-bit keys.
#include "launch.h"
#include "score16.hip"

#ifndef PALU_SCORE_FLAT
#define PALU_SCORE_FLAT 0
#endif

namespace palu {

namespace {
constexpr bool kFlat = PALU_SCORE_FLAT != 0;

template <typename T, int NK>
ScoreFn score16q_fn_n(int nq) {
  if (nq <= 2) return score16_kernel<T, NK, 1, 2, 0, kFlat>;
  if (nq <= 4) return score16_kernel<T, NK, 1, 4, 0, kFlat>;
  return score16_kernel<T, NK, 1, 8, 0, kFlat>;
}
template <typename T>
ScoreFn score16q_fn_t(int rc, int nq) {
  switch (rc) {
    case 1: return score16q_fn_n<T, 2>(nq);
    case 2: return score16q_fn_n<T, 3>(nq);
    case 3: return score16q_fn_n<T, 4>(nq);
    case 4: return score16q_fn_n<T, 5>(nq);
    case 5: return score16q_fn_n<T, 6>(nq);
    case 6: return score16q_fn_n<T, 7>(nq);
    case 7: return score16q_fn_n<T, 8>(nq);
    default: return nullptr;
  }
}

}  // namespace

template <>
ScoreFn score16q_fn<kFlat>(int act, int rc, int nq) {
  return act == PALU_F16 ? score16q_fn_t<F16>(rc, nq) : score16q_fn_t<BF16>(rc, nq);
}
// 4-bit key latents (ranks 128 and 256: whole quantization blocks), one query per head or several per key/value head
namespace {
template <int NK>
ScoreFn score16q4_fn_n(int nq, int lg) {
  if (nq == 1) {
    if constexpr (NK <= 4) { if (lg == 2) return score16_kernel<F16, NK, 4, 1, 4, kFlat>; }
    return lg == 1 ? score16_kernel<F16, NK, 2, 1, 4, kFlat> : score16_kernel<F16, NK, 1, 1, 4, kFlat>;
  }
  if (nq <= 2) return score16_kernel<F16, NK, 1, 2, 4, kFlat>;
  if (nq <= 4) return score16_kernel<F16, NK, 1, 4, 4, kFlat>;
  return score16_kernel<F16, NK, 1, 8, 4, kFlat>;
}
}  // namespace
template <>
ScoreFn score16q4_fn<kFlat>(int rc, int nq, int lg) { return rc == 3 ? score16q4_fn_n<4>(nq, lg) : (rc == 7 ? score16q4_fn_n<8>(nq, lg) : nullptr); }

}  // namespace palu
