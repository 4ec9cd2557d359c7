// step2d_sub_f32c.hip -- FP32 2D pass with several sub-steps, nv = 65.
#include "step2d_sub.h"

namespace lat {
hipError_t step2d_sub_f32_c(const StepArgs& a, hipStream_t s) {
  return launch_step2d_sub_nv<float, 65, 16, 8>(a, s);
}
}  // namespace lat
