// step2d_sub.hip -- the rules of the 2D passes with several sub-steps (all
// types): how many sub-steps a pass takes, and when a pass goes in two halves.
#include <math.h>

#include "step2d_sub.h"

namespace lat {
hipError_t step2d_sub_f64(const StepArgs& a, hipStream_t s);
hipError_t step2d_sub_f32_a(const StepArgs& a, hipStream_t s);
hipError_t step2d_sub_f32_b(const StepArgs& a, hipStream_t s);
hipError_t step2d_sub_f32_c(const StepArgs& a, hipStream_t s);

namespace {

// Parts of the small shape (0: no kernel).  The other counts of the 2D passes
// (FP32 3, 7, 11, 15 and 19, FP64 3) have none built and keep a pass per
// sub-step; shared passes were not measured there.
int sub_parts(int nv, int f64) {
  switch (nv) {
    case 5: return 2;
    case 9: return f64 ? 4 : 2;
    case 13: case 21: return f64 ? 0 : 4;
    case 17: return f64 ? 8 : 4;
    case 25: return f64 ? 0 : 8;
    case 33: return f64 ? 16 : 8;
    case 65: return f64 ? 0 : 16;
    default: return 0;
  }
}

}  // namespace

bool step2d_sub_large(int nv, int64_t pitch, int f64) {
  return !f64 && (int64_t)nv * nv * pitch * 4 > (128ll << 20);
}

// How many of `left` sub-steps the next pass takes.  Measured against a pass
// per sub-step with the shapes of step2d.h at their start (us per step of 2,
// 3, 4 sub-steps, Koren unless said):
//   Small lattices (all wavefronts run at once, a pass is one wavefront's
//   chain of rows): 64 x 48 x 33^2 84.6, 125.8, 167.1 -> 31.4, 34.3, 37.2;
//   100 x 90 x 17^2 47.5, 70.1, 92.5 -> 22.4, 26.3, 29.8; 64 x 48 x 17^2 FP64
//   43.4, 63.8, 84.2 -> 23.3, 27.2, 30.8.  Past 8000 wavefronts (2500 in FP64)
//   the stages compete for the compute units: 256^2 x 17^2 (8192) 52.8 ->
//   56.5, 210 x 150 x 17^2 FP64 (12150) 123 -> 170.
//   FP64 upwind (little arithmetic to compete for) gains at every size:
//   343 x 394 x 17^2 334, 495, 661 -> 205, 274, 369; 160 x 128 x 33^2 167,
//   248, 329 -> 137, 161, 190; 400 x 300 x 9^2 53, 79, 103 -> 37, 55, 71,
//   and with four stages 82, so up to three below 17^2.
//   Under Koren the stages have to beat the small shapes of step2d.h, which
//   spread a site's row over more lanes (a pass per sub-step in them against
//   shared passes, 2 steps): 272 x 199 x 17^2 (3383 wavefronts), 2 sub-steps
//   1.09 times longer, 192 x 135 x 25^2 (3240) 1.13, 277 x 213 x 13^2 (3834),
//   3 sub-steps 1.06; but 240 x 182 x 17^2 (2730) 0.89, 176 x 124 x 25^2
//   (2728) 0.91: up to 3000 while the state is in their range (100 MB). At
//   21^2 a lane holds six cells, and the stages lose from 1140 wavefronts on:
//   160 x 114, 2 and 3 sub-steps 1.12 and 1.19; 224 x 161 256 us a step with
//   a pass per sub-step before those shapes, 156 with them, 235 shared; at
//   744 wavefronts 0.68, 0.87, and past 3000 again 0.72.
//   Large lattices, bound by memory: FP32 only (FP64 Koren is bound by its
//   arithmetic).  65^2, 256^2 sites: 834, 1238, 1646 -> 737, 1272, 1359;
//   33^2, 512^2 sites: 835, 1249, 1665 -> 737, 1474, 1632; upwind 823, 1238,
//   1649 -> 559, 1008, 1097.  Three stages of two wavefronts leave two of the
//   four SIMDs with half the work, and four are no better than two twice
//   under Koren below 65^2.  In one wavefront per stage: 400 x 300 x 17^2
//   151, 224, 301 -> 101, 157, 227, upwind 136, 204, 274 -> 76, 102, 132.
//   Past 256 MB under Koren (sub_koren_past), 2 sub-steps: 512^2 x 17^2 232 ->
//   246, 512^2 x 21^2 381 -> 416, 2432 x 1860 x 5^2 (452 MB) 350 -> 388, 851
//   MB 1.04 times; but 9^2 0.59 to 0.76 times at 300 to 1100 MB, 13^2 0.83 to
//   1.03.
int step2d_sub_take(const lattice_dims& d, int64_t left) {
  const int P = sub_parts(d.nv, d.f64);
  if (P == 0 || left < 2) return 1;
  int64_t most;
  const int64_t bytes = (int64_t)d.nv * d.nv * d.pitch * (d.f64 ? 8 : 4);
  if (step2d_sub_large(d.nv, d.pitch, d.f64)) {
    most = !d.koren || d.nv >= 65 ? kSubMax
           : bytes > (256ll << 20) && !sub_koren_past(d.nv) ? 1 : 2;
    if (d.nv >= 25) return left >= 4 && most == 4 ? 4 : 2;
  } else {
    const int64_t S = 64 / P;
    const int64_t waves = (d.nx + S - 1) / S * d.ny;
    most = (d.f64 ? 2500 : 8000) / waves;
    if (d.koren && !d.f64 && bytes <= 100000000) {
      if (waves > 3000 && d.nv != 21) most = 1;
      if (waves > 800 && waves <= 3000 && d.nv == 21) most = 1;
    }
    if (d.f64 && !d.koren && most < kSubMax) most = d.nv >= 17 ? kSubMax : 3;
    if (most > kSubMax) most = kSubMax;
  }
  if (most < 2) return 1;
  const int64_t passes = (left + most - 1) / most;
  return (int)((left + passes - 1) / passes);
}

// A call of an odd number of passes starts from a copy of the state in the
// twin.  Where the first pass takes several sub-steps it can go in two halves
// instead (1 + 1, 2 + 1, 2 + 2): one more pass and no copy.  The copy grows
// with the state; the pass of a small lattice is a chain of nv + 3 rows, each
// longer with nv.  Measured (one step, Koren and 2 sub-steps unless said, us,
// copy against two halves; the line 250 kB nv^1.5 was fitted to 896 such
// pairs of nv 5 to 65 and 2 to 1100 MB, of which it misses the better one by
// 1 % on average):
//   below it  62 x 47 x 13^2 (2 MB) 15.2, 21.2; 57 x 42 x 25^2 (6 MB) 27.1,
//             37.3; 64 x 42 x 65^2 (45 MB) 79.2, 91.5, 4 sub-steps 87.8, 116
//   near it   155 x 119 x 9^2 (6 MB) 18.3, 19.8; 134 x 103 x 17^2 (16 MB)
//             30.5, 32.8, 4 sub-steps 54.3, 43.6; 109 x 84 x 33^2 (40 MB)
//             51.1, 54.9, 4 sub-steps 0.93 times
//   above it  281 x 215 x 17^2 (70 MB) 74, 54; 256 x 197 x 33^2 (220 MB) 259,
//             196; 1408 x 1074 x 5^2 (151 MB) 175, 124; 768 x 581 x 25^2 (1.1
//             GB) 1323, 923, upwind 989, 911; 304 x 223 x 65^2 (1.1 GB) 1285,
//             1030, 4 sub-steps 1968, 1564; FP64 upwind 240 x 182 x 17^2 (101
//             MB) 80.6, 66.7; but 130 x 100 x 65^2 (three ragged tiles a row)
//             274, 342
// Two exceptions in FP32.  Between 100 MB, where the small shapes of step2d.h
// end, and 128 MB a single pass is long for its size: 176 x 132 x 33^2 99.8,
// 172 (99.5 MB: 99.1, 81.7).  Past 128 MB two upwind sub-steps take hardly
// longer than one, and a pass longer than the copy unless its rows end on
// 64-byte sectors: 212 x 162 x 33^2 149, 169; 559 x 429 x 25^2 560, 632; but
// 512 x 382 x 17^2 210, 189; 256 x 197 x 33^2 209, 191.
bool step2d_sub_cut(const lattice_dims& d, int64_t nsub) {
  const int take = step2d_sub_take(d, nsub);
  if (take < 2) return false;
  const size_t elem = d.f64 ? 8 : 4;
  const double bytes = (double)d.nv * d.nv * d.pitch * elem;
  if (!d.f64 && bytes > 1e8) {
    if (!step2d_sub_large(d.nv, d.pitch, d.f64)) return false;
    StepArgs a = {};
    a.nx = d.nx;
    a.pitch = d.pitch;
    if (!d.koren && take == 2 && d.nv >= 9 && !step2d_aligned(a, elem))
      return false;
  }
  return bytes >= 2.5e5 * d.nv * sqrt((double)d.nv);
}

hipError_t launch_step2d_sub(const StepArgs& a, hipStream_t s) {
  if (sub_parts(a.nv, a.f64) == 0 || a.nx < 1 || a.ny < 1)
    return hipErrorInvalidValue;
  if (a.f64) return step2d_sub_f64(a, s);
  if (a.nv <= 21) return step2d_sub_f32_a(a, s);
  if (a.nv <= 33) return step2d_sub_f32_b(a, s);
  return step2d_sub_f32_c(a, s);
}

}  // namespace lat
