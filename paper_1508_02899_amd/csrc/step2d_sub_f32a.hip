// step2d_sub_f32a.hip -- FP32 2D passes with several sub-steps, nv = 5..21.
#include "step2d_sub.h"

namespace lat {
hipError_t step2d_sub_f32_a(const StepArgs& a, hipStream_t s) {
  switch (a.nv) {
    case 5: return launch_step2d_sub_nv<float, 5, 2, 0>(a, s);
    case 9: return launch_step2d_sub_nv<float, 9, 2, 0>(a, s);
    case 13: return launch_step2d_sub_nv<float, 13, 4, 0>(a, s);
    case 17: return launch_step2d_sub_nv<float, 17, 4, 0>(a, s);
    case 21: return launch_step2d_sub_nv<float, 21, 4, 0>(a, s);
    default: return hipErrorInvalidValue;
  }
}
}  // namespace lat
