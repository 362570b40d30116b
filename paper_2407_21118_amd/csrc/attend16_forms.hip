// Instantiations of the attention kernel (attend16.hip): one query per head, runs in one sequence or (PALU_SCORE_FLAT) through all; or (PALU_ATTEND_SHARED) several
// queries per key/value head (2: units of at most four query rows).
#include "launch.h"
#include "attend16.hip"

#ifndef PALU_ATTEND_SHARED
#define PALU_ATTEND_SHARED 0
#endif
#ifndef PALU_SCORE_FLAT
#define PALU_SCORE_FLAT 0
#endif

namespace palu {

namespace {
constexpr bool kFlat = PALU_SCORE_FLAT != 0;
}

#if !PALU_ATTEND_SHARED
namespace {
template <typename T, int NK>
AttendFn attend16_fn_g(int lg) {
  if constexpr (NK <= 2) { if (lg == 2) return attend16_kernel<T, NK, 4, 1, kFlat, 2>; }
  if constexpr (NK <= 4) { if (lg == 1) return attend16_kernel<T, NK, 2, 1, kFlat, 2>; }
  return lg == 0 ? attend16_kernel<T, NK, 1, 1, kFlat, 2> : nullptr;
}
template <typename T>
AttendFn attend16_fn_t(int rc, int lg) {
  switch (rc) {
    case 1: return attend16_fn_g<T, 2>(lg);
    case 2: return attend16_fn_g<T, 3>(lg);
    case 3: return attend16_fn_g<T, 4>(lg);
    case 4: return attend16_fn_g<T, 5>(lg);
    case 5: return attend16_fn_g<T, 6>(lg);
    case 6: return attend16_fn_g<T, 7>(lg);
    case 7: return attend16_fn_g<T, 8>(lg);
    default: return nullptr;
  }
}
}  // namespace

template <>
AttendFn attend16_fn<kFlat>(int act, int rc, int lg) { return act == PALU_F16 ? attend16_fn_t<F16>(rc, lg) : attend16_fn_t<BF16>(rc, lg); }
#else
namespace {
constexpr bool kFew = PALU_ATTEND_SHARED == 2;
template <typename T, int NK>
AttendFn attend16q_fn_n(int nq) {
  if (nq <= 2) return attend16_kernel<T, NK, 1, 2, kFlat, kFew ? 2 : 4>;
  if (nq <= 4) return attend16_kernel<T, NK, 1, 4, kFlat, kFew ? 2 : 8>;
  if constexpr (!kFew) return attend16_kernel<T, NK, 1, 8, kFlat, 8>;
  return nullptr;
}
template <typename T>
AttendFn attend16q_fn_t(int rc, int nq) {
  switch (rc) {
    case 1: return attend16q_fn_n<T, 2>(nq);
    case 2: return attend16q_fn_n<T, 3>(nq);
    case 3: return attend16q_fn_n<T, 4>(nq);
    case 4: return attend16q_fn_n<T, 5>(nq);
    case 5: return attend16q_fn_n<T, 6>(nq);
    case 6: return attend16q_fn_n<T, 7>(nq);
    case 7: return attend16q_fn_n<T, 8>(nq);
    default: return nullptr;
  }
}
}  // namespace

template <>
AttendFn attend16q_fn<kFew>(int act, int rc, int nq) { return act == PALU_F16 ? attend16q_fn_t<F16>(rc, nq) : attend16q_fn_t<BF16>(rc, nq); }
#endif

}  // namespace palu
