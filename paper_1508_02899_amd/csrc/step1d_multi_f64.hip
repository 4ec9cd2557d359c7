// step1d_multi_f64.hip -- FP64 instantiations of the several-steps pass.
#include "step1d_multi.h"

namespace lat {
hipError_t launch_step1d_multi_f64(const StepArgs& a, int nsteps,
                                   int64_t step0, int64_t u_hold,
                                   hipStream_t s) {
  return launch_multi_t<double>(a, nsteps, step0, u_hold, s);
}
}  // namespace lat
