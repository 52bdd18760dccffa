// Radix-2 forward procedure for K <= 7, exchanges in the vector ALU: float16
// soft values.
#include "mivit_fwd_rot.h"

namespace mivit {
hipError_t launch_rot_f16(MV_ROT_ARGS) { return rot_launch<2, 2>(K, beta, MV_ROT_PASS); }
}  // namespace mivit
