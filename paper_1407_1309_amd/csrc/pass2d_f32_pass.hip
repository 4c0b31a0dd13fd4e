// pass2d_f32_pass.hip -- FP32 instances of the 2-D single pass (pass2d.hpp)
// of a later pass.
#include "pass2d.hpp"

namespace mp {

template hipError_t pass2d_go<float, false>(const PassArgs<float> &);

}  // namespace mp
