// Instantiations of the general score kernel (score.hip) that are picked at run time: low-bit keys, fp16 shared keys.
#include "launch.h"
#include "score.hip"

namespace palu {

namespace {

// 3- and 2-bit key latents: one group per workgroup, 8 wavefronts up to rank 256, 4 half-head wavefronts above
template <int NKS>
ScoreFn score_fn_lowbit_n() {
  if constexpr (NKS > 16) return score_kernel<F16, NKS, 2, 1, 4, true, 0, true>;
  else return score_kernel<F16, NKS, 2, 1, 8, true, 0, true>;
}
}  // namespace

ScoreFn score_fn_lowbit(int rc) {
  switch (rc) {
    case 0: return score_fn_lowbit_n<2>();
    case 1: return score_fn_lowbit_n<4>();
    case 2: return score_fn_lowbit_n<6>();
    case 3: return score_fn_lowbit_n<8>();
    case 4: return score_fn_lowbit_n<10>();
    case 5: return score_fn_lowbit_n<12>();
    case 6: return score_fn_lowbit_n<14>();
    case 7: return score_fn_lowbit_n<16>();
    case 8: return score_fn_lowbit_n<18>();
    case 9: return score_fn_lowbit_n<20>();
    case 10: return score_fn_lowbit_n<22>();
    case 11: return score_fn_lowbit_n<24>();
    case 12: return score_fn_lowbit_n<26>();
    case 13: return score_fn_lowbit_n<28>();
    case 14: return score_fn_lowbit_n<30>();
    default: return score_fn_lowbit_n<32>();
  }
}

namespace {

// shared-key form (several queries per key/value head): fp16 latents, ranks up to 256, 8 wavefronts, up to 16 queries
// QP = 1: at most 4 queries per key/value head, QP = 2: at most 16
template <int QP>
ScoreFn score_fn_shared_t(int rc) {
  switch (rc) {
    case 0: return score_kernel<F16, 2, 2, 1, 8, false, QP>;
    case 1: return score_kernel<F16, 4, 2, 1, 8, false, QP>;
    case 2: return score_kernel<F16, 6, 2, 1, 8, false, QP>;
    case 3: return score_kernel<F16, 8, 2, 1, 8, false, QP>;
    case 4: return score_kernel<F16, 10, 2, 1, 8, false, QP>;
    case 5: return score_kernel<F16, 12, 2, 1, 8, false, QP>;
    case 6: return score_kernel<F16, 14, 2, 1, 8, false, QP>;
    default: return score_kernel<F16, 16, 2, 1, 8, false, QP>;
  }
}

}  // namespace

ScoreFn score_fn_shared(int rc, bool four) { return four ? score_fn_shared_t<1>(rc) : score_fn_shared_t<2>(rc); }

}  // namespace palu
