// tap_mom.hip -- the moment convolutions of setup on the direct tap kernels.
#include "tap_list.hpp"

namespace fcrkpm {
FC_TAP_MOM(FC_TAP_BUILD)
}  // namespace fcrkpm
