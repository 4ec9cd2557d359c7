// step1d_multi.hip -- FP32 instantiations of the several-steps pass and the
// rule that picks it.
#include "step1d_multi.h"

namespace lat {

hipError_t launch_step1d_multi_f64(const StepArgs& a, int nsteps,
                                   int64_t step0, int64_t u_hold,
                                   hipStream_t s);

// The recomputed halo costs more the more the update weighs against a launch:
// nsub sub-steps, twice that in FP64, and the fuller the chip is.  Measured
// against a launch per step (time ratios at 33 velocities, the closest ones):
//   up to   8192 sites (at most 256 workgroups): FP64 nsub 5 1.16, nsub 10
//           1.05; FP32 nsub 10 1.30
//   up to  16384: FP64 nsub 3 1.28, nsub 5 1.02; FP32 nsub 5 1.54
//   up to  32768: FP64 nsub 1 1.21, nsub 2 0.93; FP32 nsub 3 1.29, nsub 5 1.10
//   up to  65536: FP64 nsub 1 0.89; FP32 nsub 1 1.28, nsub 3 1.02
bool step1d_multi_lattice(int nv, int64_t nx, int nsub, int f64) {
  if (multi_parts(nv) == 0 || nx < 1) return false;
  const int64_t weight = (int64_t)nsub * (f64 ? 2 : 1);
  const int64_t most = weight <= 1   ? 65536
                       : weight <= 3 ? 32768
                       : weight <= 8 ? 16384
                       : weight <= 10 ? kMultiSmall : 0;
  return nx <= most;
}

int step1d_multi_steps(int nv, int64_t nx, int shift, int nsub, int f64) {
  if (shift < 1 || shift > 64 || !step1d_multi_lattice(nv, nx, nsub, f64))
    return 1;
  const int t = nx <= kMultiSmall ? multi_steps<32>(nv, shift)
                                  : multi_steps<64>(nv, shift);
  return t < 1 ? 1 : t;
}

hipError_t launch_step1d_multi(const StepArgs& a, int nsteps, int64_t step0,
                               int64_t u_hold, hipStream_t s) {
  if (nsteps < 1 ||
      nsteps > step1d_multi_steps(a.nv, a.nx, a.shift, a.nsub_inline, a.f64))
    return hipErrorInvalidValue;
  return a.f64 ? launch_step1d_multi_f64(a, nsteps, step0, u_hold, s)
               : launch_multi_t<float>(a, nsteps, step0, u_hold, s);
}

}  // namespace lat
