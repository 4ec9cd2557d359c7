// step2d_sub.h -- one streaming pass with several collision sub-steps for 2D
// lattices (gfx950): the row-streaming update of step2d.h with the sub-steps
// as a pipeline of wavefronts.
//
// A sub-step of its own is a pass over the whole state.  Here the wavefronts
// of a workgroup form ns stages of WPS wavefronts over the same G = WPS S
// sites: stage 0 loads the rows (pulled from the source sites) and applies
// the first sub-step, stage q the sub-step q + 1 to the rows that stage
// q - 1 finished, and the rows of the last stage go to memory.  A finished
// row passes to the next stage through LDS; row t leaves a stage three rows
// after it entered, and one more for the barrier, so stage q works on row
// T - 4 q at tick T and a pass of NV + 3 + 4 (ns - 1) ticks replaces ns
// passes of NV + 3.  Every element is read once and written once per pass,
// and the bits are those of the separate passes.
//
// The Koren passes in two-wavefront stages fill the 256 registers and spill
// four of them at 65 velocities (20 bytes a lane) and three at 33 (16 bytes).
//
// Bound by the arithmetic of the Koren fluxes (upwind: by memory) where the
// lattice is large, by the latency of a tick where it is small.  256^2 sites
// x 65^2, 4 sub-steps: 1646 -> 1359 us a step (four passes at 4.4 TB/s had
// 1646); 64 x 48 sites x 33^2, 4 sub-steps: 167 -> 37 us.
#pragma once

#include "step2d.h"

#pragma clang fp contract(off)

namespace lat {

constexpr int kSubMax = 4;  // stages of a workgroup

// Whether two Koren sub-steps share a pass past 256 MB (measured per shape:
// step2d_sub_take).
constexpr bool sub_koren_past(int nv) {
  return nv != 5 && nv != 17 && nv != 21;
}

template <typename T, int NV, int P, bool KOREN, bool INTERIOR, bool FIRST,
          int WPS, bool NT>
__device__ __forceinline__ void step2d_sub_wave(
    const T* __restrict__ fin, T* __restrict__ fout, const T* __restrict__ u,
    const int* __restrict__ flag, T* __restrict__ stage, int nx, int ny,
    size_t pitch, int shift, int xstep, int xoff0, int ystep, int yoff0,
    T alpha_scale, T beta, T D, int xb, int w, int y, int q, int ns) {
  using K = Step2D<T, NV, P, KOREN>;
  using O = OutStage<T, NV, P, WPS>;
  constexpr int W = K::W, S = K::S, H = K::H, G = O::G;
  const int lane = (int)threadIdx.x & 63;
  const int p = lane / S;
  const int sl = lane - p * S;
  const int x0 = xb + w * S;  // first site of this wavefront
  // outside the row: duplicate its first or last site
  const int x = max(0, min(x0 + sl, nx - 1));
  const bool first = p == 0, last = p == P - 1;
  const int lane_l = lane - S, lane_r = lane + S;
  const int jx0 = p * (W - 1);  // first vx cell of this lane

  const size_t nxy = (size_t)nx * (size_t)ny;
  const size_t rowpitch = (size_t)NV * pitch;
  const T ax = u[(size_t)y * nx + x] * alpha_scale;
  const T ay = u[nxy + (size_t)y * nx + x] * alpha_scale;
  const int stop = *flag;

  T nxp[W + 2], nxm[W + 2];
#pragma unroll
  for (int i = 0; i < W + 2; ++i) {
    const T nu = fma_t(-beta, (T)(jx0 + i - 1 - H), ax);
    nxp[i] = pos(nu);
    nxm[i] = neg(nu);
  }

  // stage 0: byte offsets of the cells of one vy row, as in step2d_tile
  uint32_t koff[FIRST && !INTERIOR ? W : 1];
  uint32_t cell_stride = 0;
  const T* fbase = fin;
  if constexpr (FIRST && INTERIOR) {
    koff[0] = (uint32_t)(((size_t)jx0 * (pitch - shift) + (size_t)sl) *
                         sizeof(T));
    cell_stride = (uint32_t)((pitch - shift) * sizeof(T));
    fbase = fin + x0 + (size_t)shift * H;
  } else if constexpr (FIRST) {
    int xs = x + xoff0;
    if (xs >= nx) xs -= nx;
    for (int k = 0; k < jx0; ++k) {
      xs -= xstep;
      if (xs < 0) xs += nx;
    }
#pragma unroll
    for (int i = 0; i < W; ++i) {
      koff[i] = (uint32_t)(((size_t)(jx0 + i) * pitch + (size_t)xs) *
                           sizeof(T));
      xs -= xstep;
      if (xs < 0) xs += nx;
    }
  }
  int ys = y + yoff0;  // row t = 0 comes from (y + shift*H) mod ny
  if (ys >= ny) ys -= ny;
  // the next row (stage 0: rows are asked for in order, each once)
  const int cell0 = jx0 * O::STRIDE + w * S + sl;
  auto load_row = [&](int t, T (&c)[W]) {
    if constexpr (FIRST) {
      const T* src = fbase + (size_t)t * rowpitch + (size_t)ys * nx;
      uint32_t lo = koff[0];
      if (INTERIOR) asm volatile("" : "+v"(lo));
#pragma unroll
      for (int i = 0; i < W; ++i)
        c[i] = INTERIOR ? row_load(src, (uint32_t)i * cell_stride, lo)
                        : row_load(src, 0u, koff[i]);
      int v = ys - ystep;
      ys = __builtin_amdgcn_readfirstlane(v < 0 ? v + ny : v);
    } else {
      const T* src = stage + (2 * (q - 1) + (t & 1)) * O::SIZE + cell0;
#pragma unroll
      for (int i = 0; i < W; ++i) c[i] = src[i * O::STRIDE];
    }
  };

  // End of a tick: the rows written in it become visible, and every thread
  // stores its share of the row that the last stage finished in it: planes
  // fj0 + PR k of site fs.
  const int tid = (int)threadIdx.x;
  const int PR = ns * P;
  const int fj0 = tid / G, fs = tid - fj0 * G;
  const int fx = max(0, min(xb + fs, nx - 1));
  const uint32_t flane =
      (uint32_t)(((size_t)fj0 * pitch + (size_t)(fx - xb)) * sizeof(T));
  T* const frow0 = fout + ((int64_t)y * nx + xb);
  const uint32_t slot_bytes = (uint32_t)(pitch * sizeof(T));
  const T* const fin_stage =
      stage + 2 * (ns - 1) * O::SIZE + fj0 * O::STRIDE + fs;
  constexpr int KM = (NV + 2 * P - 1) / (2 * P);  // rounds with two stages
  auto tick_end = [&](int tick) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    const int r = tick - 4 * (ns - 1) - 3;
    if (r < 0) return;
    const T* sb = fin_stage + (r & 1) * O::SIZE;
    T* orow = frow0 + (size_t)r * rowpitch;
    T v[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k)
      v[k] = fj0 + PR * k < NV ? sb[k * PR * O::STRIDE] : T(0);
#pragma unroll
    for (int k = 0; k < KM; ++k)
      row_store_if<NT>(orow, (uint32_t)(k * PR) * slot_bytes, flane, v[k],
                       fj0 + PR * k < NV);
  };

  YState<T, W> st;
#pragma unroll
  for (int i = 0; i < W; ++i) {
    st.gp1[i] = st.dpp1[i] = st.gm1[i] = st.em1[i] = st.Fp1[i] =
        st.acc2[i] = st.c1[i] = st.a3[i] = st.del3[i] = T(0);
  }
  T* const dst = stage + 2 * q * O::SIZE + cell0;
  // kind: -1 for an edge row, else the steady row's skip mode
  auto run_row = [&](auto kind, int t, const T (&c)[W]) {
    constexpr int KIND = decltype(kind)::value;
    constexpr bool STEADY = KIND >= 0;
    T* const o = dst + ((t + 1) & 1) * O::SIZE;  // row t - 3
    K::template row<STEADY, STEADY ? KIND : 0>(
        t, c, st, nxp, nxm, ay, beta, D, first, last, lane_l, lane_r,
        [&](int i, T v) { o[i * O::STRIDE] = v; });
    tick_end(t + 4 * q);
  };
  using edge_t = std::integral_constant<int, -1>;
  auto skip_gm = [&](int t) {
    return beta >= T(0) && __all(fma_t(-beta, (T)(t + 1 - H), ay) >= T(0));
  };
  auto skip_gp = [&](int t) {
    return beta >= T(0) && __all(fma_t(-beta, (T)(t - 1 - H), ay) <= T(0));
  };

  T bufA[W], bufB[W];
  if constexpr (FIRST) {
    load_row(0, bufA);
    load_row(1, bufB);
    asm volatile("" ::: "memory");
    if (stop != 0) return;  // uniform over the grid
    run_row(edge_t(), 0, bufA);
    load_row(2, bufA);
    run_row(edge_t(), 1, bufB);
    if (NV > 3) load_row(3, bufB);
    run_row(edge_t(), 2, bufA);
  } else {
    if (stop != 0) return;
    for (int k = 0; k < 4 * q; ++k) tick_end(k);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      load_row(t, bufA);
      run_row(edge_t(), t, bufA);
    }
  }
  // steady pair (t, t+1); stage 0: row t is in bufB
  auto pair = [&](auto mode, int t, bool load2) {
    if constexpr (FIRST) {
      load_row(t + 1, bufA);
      run_row(mode, t, bufB);
      if (load2) load_row(t + 2, bufB);
      run_row(mode, t + 1, bufA);
    } else {
      load_row(t, bufA);
      run_row(mode, t, bufA);
      load_row(t + 1, bufA);
      run_row(mode, t + 1, bufA);
    }
  };
  if (NV >= 7) {
    pair(std::integral_constant<int, 0>(), 3, true);
    int t = 5;
#pragma unroll 1
    for (; t <= NV - 4 && skip_gm(t); t += 2)
      pair(std::integral_constant<int, 1>(), t, true);
#pragma unroll 1
    for (; t <= NV - 4 && !skip_gp(t); t += 2)
      pair(std::integral_constant<int, 0>(), t, true);
#pragma unroll 1
    for (; t <= NV - 4; t += 2)
      pair(std::integral_constant<int, 2>(), t, true);
    pair(std::integral_constant<int, 0>(), NV - 2, false);
  } else if (NV == 5) {
    pair(std::integral_constant<int, 3>(), 3, false);
  }
  run_row(edge_t(), NV, bufB);
  run_row(edge_t(), NV + 1, bufB);
  run_row(edge_t(), NV + 2, bufB);
  for (int k = NV + 3 + 4 * q; k < NV + 3 + 4 * (ns - 1); ++k) tick_end(k);
}

template <typename T, int NV, int P, bool KOREN, bool NT, int WPS>
__global__ __launch_bounds__(64 * WPS * kSubMax, 2) void k_step2d_sub(
    const T* __restrict__ fin, T* __restrict__ fout, const T* __restrict__ u,
    const int* __restrict__ flag, int nx, int ny, int64_t pitch, int shift,
    int xstep, int xoff0, int ystep, int yoff0, T alpha_scale, T beta, T D,
    int ngx, int nblocks, int rows, int sector, int ns) {
  using O = OutStage<T, NV, P, WPS>;
  constexpr int S = 64 / P;
  constexpr int H = (NV - 1) / 2;
  __shared__ T stage[2 * kSubMax * O::SIZE];
  const int b = xcd_rows(blockIdx.x, nblocks, ngx * rows);
  const int y = b / ngx;
  const int xg = b - y * ngx;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int q = wv / WPS, w = wv - q * WPS;
  const int xb = xg * O::G - ((y * nx) & sector);  // the tile's first site
  const int x0 = xb + w * S;
  const bool interior = x0 + S <= nx && x0 - shift * H >= 0 &&
                        x0 + S - 1 + shift * H <= nx - 1;
  if (q > 0)
    step2d_sub_wave<T, NV, P, KOREN, true, false, WPS, NT>(
        fin, fout, u, flag, stage, nx, ny, (size_t)pitch, shift, xstep, xoff0,
        ystep, yoff0, alpha_scale, beta, D, xb, w, y, q, ns);
  else if (interior)
    step2d_sub_wave<T, NV, P, KOREN, true, true, WPS, NT>(
        fin, fout, u, flag, stage, nx, ny, (size_t)pitch, shift, xstep, xoff0,
        ystep, yoff0, alpha_scale, beta, D, xb, w, y, 0, ns);
  else
    step2d_sub_wave<T, NV, P, KOREN, false, true, WPS, NT>(
        fin, fout, u, flag, stage, nx, ny, (size_t)pitch, shift, xstep, xoff0,
        ystep, yoff0, alpha_scale, beta, D, xb, w, y, 0, ns);
}

template <typename T, int NV, int P, int WPS, bool BIG>
hipError_t launch_step2d_sub_shape(const StepArgs& a, hipStream_t s) {
  constexpr int G = OutStage<T, NV, P, WPS>::G;
  if (!step2d_offsets_fit(NV, a.pitch, sizeof(T)) || a.pitch < a.nx * a.ny ||
      a.nsub_inline < 2 || a.nsub_inline > kSubMax)
    return hipErrorNotSupported;
  const int nx = (int)a.nx, ny = (int)a.ny;
  const int H = (NV - 1) / 2;
  const int ngx = (nx + G - 1) / G;
  const int64_t nb = (int64_t)ngx * ny;
  if (nb > 0x7FFFFFFF) return hipErrorInvalidValue;
  const int nblocks = (int)nb;
  const int xstep = a.shift % nx;
  const int xoff0 = (int)(((int64_t)a.shift * H) % nx);
  const int ystep = a.shift % ny;
  const int yoff0 = (int)(((int64_t)a.shift * H) % ny);
  const T as = (T)a.alpha_scale, be = (T)a.beta, D = (T)a.D;
  const bool nt = step2d_nt(a, NV, sizeof(T));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(64 * WPS * a.nsub_inline),
                       0, s, (const T*)a.fin, (T*)a.fout, (const T*)a.u,
                       a.flag, nx, ny, a.pitch, a.shift, xstep, xoff0, ystep,
                       yoff0, as, be, D, ngx, nblocks,
                       step2d_rows(a, sizeof(T)),
                       step2d_sector(a, G, sizeof(T)), a.nsub_inline);
  };
  if (BIG && nt) {
    constexpr bool past = BIG && sub_koren_past(NV);
    if (a.koren && !past) return hipErrorNotSupported;  // one sub-step a pass
    if (a.koren)
      go(k_step2d_sub<T, NV, P, true, past, WPS>);
    else
      go(k_step2d_sub<T, NV, P, false, BIG, WPS>);
  } else {
    if (a.koren)
      go(k_step2d_sub<T, NV, P, true, false, WPS>);
    else
      go(k_step2d_sub<T, NV, P, false, false, WPS>);
  }
  return hipGetLastError();
}

// The two shapes of a lattice: SMALL in PS parts with one wavefront per
// stage, and from nv 25 on (FP32) LARGE in PL parts with two.
template <typename T, int NV, int PS, int PL>
hipError_t launch_step2d_sub_nv(const StepArgs& a, hipStream_t s) {
  if constexpr (PL > 0) {
    if (step2d_sub_large(a.nv, a.pitch, a.f64))
      return launch_step2d_sub_shape<T, NV, PL, 2, true>(a, s);
    return launch_step2d_sub_shape<T, NV, PS, 1, false>(a, s);
  } else {
    return launch_step2d_sub_shape<T, NV, PS, 1, sizeof(T) == 4>(a, s);
  }
}

}  // namespace lat
