// tap_f32.hip -- the FP32 variants of the direct tap kernels.
#include "tap_list.hpp"

namespace fcrkpm {
FC_TAP_F32(FC_TAP_BUILD)
}  // namespace fcrkpm
