// tap_f64n.hip -- the FP64 variants of u^h, the loads and the gradient force
// on the direct tap kernels.
#include "tap_list.hpp"

namespace fcrkpm {
FC_TAP_F64N(FC_TAP_BUILD)
}  // namespace fcrkpm
