// Radix-2 forward procedure for K = 8 and 9, float16 soft values.
#include "mivit_fwd_wide_float.h"

namespace mivit {
hipError_t launch_wide_f16(int K, int beta, int wpf, const DevCode* codes, const Item* items,
                           const SplitUnit* units, int n_units, const void* llr, uint64_t* surv,
                           void* metric, int32_t* end_out, int32_t* item_end, hipStream_t st) {
  return wf_launch<2>(K, beta, wpf, codes, items, units, n_units, llr, surv, metric, end_out,
                      item_end, st);
}
}  // namespace mivit
