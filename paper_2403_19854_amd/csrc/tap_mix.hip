// tap_mix.hip -- the direct tap kernels with FP32 arithmetic on FP64 fields.
#include "tap_list.hpp"

namespace fcrkpm {
FC_TAP_MIX(FC_TAP_BUILD)
}  // namespace fcrkpm
