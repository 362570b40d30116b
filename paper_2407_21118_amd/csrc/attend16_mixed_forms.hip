// Instantiations of the attention kernel over units of several key ranks (attend16.hip).
#include "launch.h"
#include "attend16.hip"

#ifndef PALU_SCORE_FLAT
#define PALU_SCORE_FLAT 0
#endif

namespace palu {

template <>
AttendFn attend16_mixed_fn<PALU_SCORE_FLAT != 0>(int act) {
  return act == PALU_F16 ? attend16_mixed_kernel<F16, PALU_SCORE_FLAT != 0> : attend16_mixed_kernel<BF16, PALU_SCORE_FLAT != 0>;
}

}  // namespace palu
