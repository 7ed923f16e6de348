// tap_cg32.hip -- the FP32 K products of CG on the direct tap kernels (with the
// direction update).
#include "tap_list.hpp"

namespace fcrkpm {
FC_TAP_CG32(FC_TAP_BUILD)
}  // namespace fcrkpm
