// pass2d_f64_donor.hip -- FP64 instances of the 2-D single pass (pass2d.hpp)
// with the donor pass folded in.
#include "pass2d.hpp"

namespace mp {

template hipError_t pass2d_go<double, true>(const PassArgs<double> &);

}  // namespace mp
