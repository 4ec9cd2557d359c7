// step2d_sub_f64.hip -- FP64 2D passes with several sub-steps.
#include "step2d_sub.h"

namespace lat {

hipError_t step2d_sub_f64(const StepArgs& a, hipStream_t s) {
  switch (a.nv) {
    case 5: return launch_step2d_sub_nv<double, 5, 2, 0>(a, s);
    case 9: return launch_step2d_sub_nv<double, 9, 4, 0>(a, s);
    case 17: return launch_step2d_sub_nv<double, 17, 8, 0>(a, s);
    default: return launch_step2d_sub_nv<double, 33, 16, 0>(a, s);
  }
}

}  // namespace lat
