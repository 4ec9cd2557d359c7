// step2d_sub_f32b.hip -- FP32 2D passes with several sub-steps, nv = 25, 33.
#include "step2d_sub.h"

namespace lat {
hipError_t step2d_sub_f32_b(const StepArgs& a, hipStream_t s) {
  switch (a.nv) {
    case 25: return launch_step2d_sub_nv<float, 25, 8, 4>(a, s);
    case 33: return launch_step2d_sub_nv<float, 33, 8, 4>(a, s);
    default: return hipErrorInvalidValue;
  }
}
}  // namespace lat
