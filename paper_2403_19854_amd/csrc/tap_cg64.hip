// tap_cg64.hip -- the FP64 K products of CG on the direct tap kernels (with the
// direction update).
#include "tap_list.hpp"

namespace fcrkpm {
FC_TAP_CG64(FC_TAP_BUILD)
}  // namespace fcrkpm
