// Radix-2 forward procedure for K <= 7: dispatch, and the kernels that
// exchange through LDS swizzles (variants 1 and 2).
#include "mivit_fwd_rot.h"

namespace mivit {

hipError_t launch_fwd_rot(int K, int beta, int dt, int mode, const DevCode* codes,
                          const Item* items, const int2* waves, int n_waves, const void* llr,
                          uint64_t* surv, void* metric, int32_t* end_out, int32_t* item_end,
                          int32_t* counter, int grid_limit, hipStream_t st) {
  if (n_waves <= 0) return hipSuccess;
  // float16 soft values: the all-VALU exchange scheme (MODE 2) only
  if (dt < 0 || dt > 2 || (dt == 2 && mode != 2)) return hipErrorInvalidValue;
  if (mode == 2)
    return dt == 0   ? launch_rot_f32(K, beta, MV_ROT_PASS)
           : dt == 1 ? launch_rot_i8(K, beta, MV_ROT_PASS)
                     : launch_rot_f16(K, beta, MV_ROT_PASS);
  if (mode == 1)
    return dt == 0 ? rot_launch<0, 1>(K, beta, MV_ROT_PASS)
                   : rot_launch<1, 1>(K, beta, MV_ROT_PASS);
  return dt == 0 ? rot_launch<0, 0>(K, beta, MV_ROT_PASS)
                 : rot_launch<1, 0>(K, beta, MV_ROT_PASS);
}

}  // namespace mivit
