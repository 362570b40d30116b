// Instantiations of the attention kernel over units of several key ranks (attend16.hip).
#include "launch.h"
#include "attend16.hip"

namespace palu {

AttendFn attend16_mixed_fn(int act) { return act == PALU_F16 ? attend16_mixed_kernel<F16> : attend16_mixed_kernel<BF16>; }

}  // namespace palu
