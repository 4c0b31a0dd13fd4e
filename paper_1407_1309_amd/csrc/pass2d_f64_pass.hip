// pass2d_f64_pass.hip -- FP64 instances of the 2-D single pass (pass2d.hpp)
// of a later pass.
#include "pass2d.hpp"

namespace mp {

template hipError_t pass2d_go<double, false>(const PassArgs<double> &);

}  // namespace mp
