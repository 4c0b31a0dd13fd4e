// resident1d_f32.hip -- FP32 instances of the 1-D steps (line1d.hpp).
#include "line1d.hpp"

namespace mp {

template hipError_t line1d_launch<float>(const LineShape &, const LineArgs<float> &, int,
                                         const float *, const float *, float *, float *,
                                         hipStream_t);

}  // namespace mp
