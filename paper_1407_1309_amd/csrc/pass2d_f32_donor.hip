// pass2d_f32_donor.hip -- FP32 instances of the 2-D single pass (pass2d.hpp)
// with the donor pass folded in.
#include "pass2d.hpp"

namespace mp {

template hipError_t pass2d_go<float, true>(const PassArgs<float> &);

}  // namespace mp
