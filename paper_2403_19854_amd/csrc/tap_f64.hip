// tap_f64.hip -- the FP64 variants of the direct tap kernels.
#include "tap_list.hpp"

namespace fcrkpm {
FC_TAP_F64(FC_TAP_BUILD)
}  // namespace fcrkpm
