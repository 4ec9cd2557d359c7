// step1d_multi.h -- several 1D time steps per launch for short lattices
// (gfx950).
//
// A short lattice (up to 8192 sites, and with few sub-steps up to 65536:
// step1d_multi_lattice) leaves the chip idle and its step is a launch: the
// host issues one every 2.9 us (8 us for the first fifty after an idle
// queue), whatever the step computes.  Here a workgroup takes G sites through
// T steps in LDS.  The mass of velocity index j moves s (j - h) cells per
// step, so G finished sites need the start values of the sites up to h s T
// away on either side: the workgroup loads G + 2 h s T sites and updates a
// region that shrinks by h s on either side per step.
// The neighbours compute the same halo sites again from the same values with
// the same operations; no workgroup waits for another.  The update is the
// split-column one (parts1d.h), bit for bit that of the one-step pass of the
// same lattice (step1d_parts.hip, or step1d.hip with the same arithmetic).
// Measured per step of a call of 200 (one launch per step before): 256 x 33
// FP64 3.7 -> 2.1 us, 256 x 17 FP32 2.8 -> 1.0, 4096 x 9 FP32 3.75 -> 0.75,
// 16384 x 33 FP32 3.4 -> 1.7, 65536 x 17 FP32 4.0 -> 2.7.  What is left is the
// update of the region by one compute unit and, per launch, one load and one
// store latency.
#pragma once

#include "lattice_internal.h"
#include "parts1d.h"

namespace lat {

// Finished sites G, sites loaded at most.  32 sites spread a short lattice
// over the most compute units; from 257 such workgroups on, 64 sites
// recompute less (16384 x 33 FP64: 4.3 us a step with 32, 2.7 with 64; 256 x
// 33 FP64: 2.2 with 32, 2.4 with 64).
template <int G>
struct MultiTile;
template <> struct MultiTile<32> {
  static constexpr int REGION = 160;
};
template <> struct MultiTile<64> {
  static constexpr int REGION = 192;
};

// Velocity lattices with a kernel and the parts of their columns (lanes of
// 3 to 6 cells; halving or doubling them changes the step by under 10 %).  11,
// 15, 19, 23, 27, 29 and 31 have none built and keep a launch per step; the
// pass was not measured there.  From 65 velocities on a region of 160 sites
// holds two steps at most, with two halo sites for each finished one and more.
constexpr int multi_parts(int nv) {
  switch (nv) {
    case 3: return 1;
    case 5: case 7: return 2;
    case 9: case 13: case 17: case 21: return 4;
    case 25: case 33: return 8;
    default: return 0;
  }
}

// Wavefronts of a workgroup: 16 where 8 would go over a region in three
// rounds, being 8 sites each (25 and 33 velocities at G = 32; us a step, 8
// against 16, 256 sites: 33 FP64 2.19, 2.14, FP32 with 3 sub-steps 2.39, 2.18;
// 25 FP64 1.87, 1.80, FP32 1.44, 1.36; but 5 FP64 0.74, 0.75, 17 FP64 1.33,
// 1.36), and for G = 64.
template <int G>
constexpr int multi_waves(int nv) {
  return G == 64 || multi_parts(nv) == 8 ? 16 : 8;
}

// Steps per launch: as many as the region allows, at most 16.
template <int G>
constexpr int multi_steps(int nv, int shift) {
  const int64_t t = (MultiTile<G>::REGION - G) /
                    (2 * (int64_t)shift * ((nv - 1) / 2));
  return t > 16 ? 16 : (int)t;
}

template <typename T, int NV, int G, bool KOREN>
__global__ __launch_bounds__(64 * multi_waves<G>(NV)) void k_step1d_multi(
    const T* __restrict__ fin, T* __restrict__ fout, const T* __restrict__ u,
    const int* __restrict__ flag, int nx, int shift, int nsub, T alpha_scale,
    T beta, T D, int nsteps, int64_t step0, int64_t u_hold, int nblocks) {
  constexpr int P = multi_parts(NV);
  constexpr int REGION = MultiTile<G>::REGION, WAVES = multi_waves<G>(NV);
  using PT = Parts1DTile<T, NV, P, WAVES>;
  constexpr int W = PT::W, S = PT::S, H = PT::H;
  constexpr int PITCH = REGION + 2;
  constexpr int TM = multi_steps<G>(NV, 1);
  __shared__ T buf[2][NV * PITCH];
  __shared__ T us[TM][REGION];
  const int stop = *flag;
  const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
  const int hs = H * shift;
  const int width = G + 2 * hs * nsteps;  // <= REGION (host)
  const int x0 = xcd_remap(blockIdx.x, nblocks) * G;
  // sites of this lane in the loaded region: lane, lane + 64, lane + 128
  constexpr int NC = (REGION + 63) / 64;
  int xs[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int i = min(lane + 64 * q, width - 1);
    int x = (x0 - hs * nsteps + i) % nx;
    xs[q] = x < 0 ? x + nx : x;
  }
  {
    constexpr int NJ = (NV + WAVES - 1) / WAVES;
    T v[NJ][NC];
#pragma unroll
    for (int a = 0; a < NJ; ++a) {
      const int j = min(w + WAVES * a, NV - 1);
#pragma unroll
      for (int q = 0; q < NC; ++q) v[a][q] = fin[(size_t)j * nx + xs[q]];
    }
    for (int k = w; k < nsteps; k += WAVES) {
      const T* const uk = u + (u_hold > 0 ? (step0 + k) / u_hold : 0) * nx;
#pragma unroll
      for (int q = 0; q < NC; ++q)
        if (lane + 64 * q < width) us[k][lane + 64 * q] = uk[xs[q]];
    }
#pragma unroll
    for (int a = 0; a < NJ; ++a) {
      const int j = w + WAVES * a;
#pragma unroll
      for (int q = 0; q < NC; ++q)
        if (j < NV && lane + 64 * q < width)
          buf[0][j * PITCH + lane + 64 * q] = v[a][q];
    }
  }
  __syncthreads();
  const int p = lane / S, sl = lane - p * S;
  const int j0 = p * (W - 1);
  for (int k = 0; k < nsteps; ++k) {
    const T* const src = buf[k & 1];
    T* const dst = buf[(k & 1) ^ 1];
    const int lo = hs * (k + 1), hi = width - lo;  // this step's region
    for (int g = lo + w * S; g < hi; g += WAVES * S) {
      const int i = min(g + sl, hi - 1);  // past the end: a real site
      const T* const col = src + j0 * PITCH + i - shift * (j0 - H);
      T c[W];
#pragma unroll
      for (int e = 0; e < W; ++e) c[e] = col[e * (PITCH - shift)];
      PT::template update<KOREN>(c, us[k][i] * alpha_scale, nsub, beta, D);
      if (g + sl < hi) {
        T* const out = dst + j0 * PITCH + i;
#pragma unroll
        for (int e = 0; e < W - 1; ++e) out[e * PITCH] = c[e];
        if (p == P - 1) out[(W - 1) * PITCH] = c[W - 1];
      }
    }
    __syncthreads();
  }
  if (stop != 0) return;
  const T* const res = buf[nsteps & 1] + hs * nsteps;
  constexpr int PL = 64 * WAVES / G;  // planes per round
  const int i = (int)threadIdx.x % G;
  if (x0 + i >= nx) return;
#pragma unroll
  for (int a = 0; a < (NV + PL - 1) / PL; ++a) {
    const int j = (int)threadIdx.x / G + PL * a;
    if (j < NV) fout[(size_t)j * nx + x0 + i] = res[j * PITCH + i];
  }
}

template <typename T, int NV, int G>
hipError_t launch_multi_g(const StepArgs& a, int nsteps, int64_t step0,
                          int64_t u_hold, hipStream_t s) {
  const int nblocks = (int)((a.nx + G - 1) / G);
  const T as = (T)a.alpha_scale, be = (T)a.beta, D = (T)a.D;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(64 * multi_waves<G>(NV)),
                       0, s, (const T*)a.fin, (T*)a.fout, (const T*)a.u, a.flag,
                       (int)a.nx, a.shift, a.nsub_inline, as, be, D, nsteps,
                       step0, u_hold, nblocks);
  };
  if (a.koren)
    go(k_step1d_multi<T, NV, G, true>);
  else
    go(k_step1d_multi<T, NV, G, false>);
  return hipGetLastError();
}

template <typename T, int NV>
hipError_t launch_multi_nv(const StepArgs& a, int nsteps, int64_t step0,
                           int64_t u_hold, hipStream_t s) {
  return a.nx <= kMultiSmall
             ? launch_multi_g<T, NV, 32>(a, nsteps, step0, u_hold, s)
             : launch_multi_g<T, NV, 64>(a, nsteps, step0, u_hold, s);
}

template <typename T>
hipError_t launch_multi_t(const StepArgs& a, int n, int64_t step0,
                          int64_t u_hold, hipStream_t s) {
  switch (a.nv) {
    case 3: return launch_multi_nv<T, 3>(a, n, step0, u_hold, s);
    case 5: return launch_multi_nv<T, 5>(a, n, step0, u_hold, s);
    case 7: return launch_multi_nv<T, 7>(a, n, step0, u_hold, s);
    case 9: return launch_multi_nv<T, 9>(a, n, step0, u_hold, s);
    case 13: return launch_multi_nv<T, 13>(a, n, step0, u_hold, s);
    case 17: return launch_multi_nv<T, 17>(a, n, step0, u_hold, s);
    case 21: return launch_multi_nv<T, 21>(a, n, step0, u_hold, s);
    case 25: return launch_multi_nv<T, 25>(a, n, step0, u_hold, s);
    case 33: return launch_multi_nv<T, 33>(a, n, step0, u_hold, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lat
