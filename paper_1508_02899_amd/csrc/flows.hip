// flows.hip -- carrier-flow synthesis on the device from Fourier mode tables
// (gfx950), so that long runs need no prestaged velocity field.
//
// The flows are the random Fourier flows of Sec. 3 (1D: a sum of modes whose
// amplitudes are redrawn or evolve as Ornstein-Uhlenbeck processes, Eq. 7)
// and the incompressible 2D flows of Sec. 4 (u = (d_y psi, -d_x psi) from a
// streamfunction).  The host draws the mode amplitudes (one table row per
// time slice); this file evaluates them on the lattice sites.  Phases are
// exact: the angle 2 pi k j / n is formed from the integer (k j) mod n.
#include <math.h>

#include "../../include/lattice.h"
#include "lattice_struct.h"

namespace lat {
namespace {

constexpr int kFlowBlock = 256;

__device__ __forceinline__ void phase(int64_t k, int64_t j, int64_t n,
                                      float* c, float* s) {
  int64_t p = (k * j) % n;
  if (p < 0) p += n;
  sincospif(2.0f * (float)p / (float)n, s, c);
}
__device__ __forceinline__ void phase(int64_t k, int64_t j, int64_t n,
                                      double* c, double* s) {
  int64_t p = (k * j) % n;
  if (p < 0) p += n;
  sincospi(2.0 * (double)p / (double)n, s, c);
}

// 1D: u[s][ix] = sum_k a_k cos(2 pi k ix / nx) + b_k sin(...), k = 1..K.
// coef[s][k-1] = (a, b).  One thread per site, one grid row per slice.
template <typename T>
__global__ __launch_bounds__(kFlowBlock) void k_flow1d(
    const float* __restrict__ coef, int K, int64_t nx, T* __restrict__ u) {
  const int64_t ix = (int64_t)blockIdx.x * kFlowBlock + threadIdx.x;
  const int64_t s = blockIdx.y;
  if (ix >= nx) return;
  const float* c = coef + (size_t)s * K * 2;
  T acc = 0;
  for (int k = 1; k <= K; ++k) {
    T cs, sn;
    phase(k, ix, nx, &cs, &sn);
    acc += (T)c[2 * (k - 1)] * cs + (T)c[2 * (k - 1) + 1] * sn;
  }
  u[(size_t)s * nx + ix] = acc;
}

// The same phase for k >= 0 with a product that fits 32 bits (no 64-bit
// division).
template <typename T>
__device__ __forceinline__ void phase_k(uint32_t k, uint32_t j, uint32_t n,
                                        T* c, T* s) {
  const uint64_t q = (uint64_t)k * j;
  const uint32_t p = (q >> 32) == 0 ? (uint32_t)q % n : (uint32_t)(q % n);
  if constexpr (sizeof(T) == 4)
    sincospif(2.0f * (float)p / (float)n, s, c);
  else
    sincospi(2.0 * (double)p / (double)n, s, c);
}

// 2D, pass 1 (along x): with E[ky][ix] = sum_kx c[ky][kx] e^{2 pi i kx ix/nx}
// and B the same sum with kx c, the rows ky and -ky (ky = 0..K; the row -0
// is left out) combined into the four real numbers that pass 2 needs:
//   W[ky][0] = -gy ky (Im E+ - Im E-),   W[ky][1] = -gy ky (Re E+ + Re E-),
//   W[ky][2] =  gx (Im B+ + Im B-),      W[ky][3] =  gx (Re B+ - Re B-)
// (gx, gy = 2 pi / (nx dx), 2 pi / (ny dx)), so that
//   u_x = d psi/dy  = sum_ky W0 cos(th) + W1 sin(th),
//   u_y = -d psi/dx = sum_ky W2 cos(th) + W3 sin(th),  th = 2 pi ky iy / ny.
// coef[s][ky + K][kx] = (re, im), kx = 0..K.  A block takes 64 sites and
// kFlowRows values of ky: the twiddles are computed once for all of them
// (they were the cost of a thread per site and row).
constexpr int kFlowRows = 4;
template <typename T>
__global__ __launch_bounds__(kFlowBlock) void k_flow2d_x(
    const float* __restrict__ coef, int K, int nx, T gx, T gy,
    T* __restrict__ W) {
  __shared__ T tw[65][64][2];
  const int l = (int)threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ix = (int)blockIdx.x * 64 + l;
  for (int k = w; k <= K; k += kFlowBlock / 64) {
    T cs, sn;
    phase_k<T>((uint32_t)k, (uint32_t)(ix < nx ? ix : 0), (uint32_t)nx, &cs,
               &sn);
    tw[k][l][0] = cs;
    tw[k][l][1] = sn;
  }
  __syncthreads();
  if (ix >= nx) return;
  const int64_t s = blockIdx.z;
  const int r0 = (int)blockIdx.y * kFlowRows;
  for (int ky = r0 + w; ky <= K && ky < r0 + kFlowRows;
       ky += kFlowBlock / 64) {
    const float* cp = coef + (((size_t)s * (2 * K + 1)) + K + ky) * (K + 1) * 2;
    const float* cm = coef + (((size_t)s * (2 * K + 1)) + K - ky) * (K + 1) * 2;
    const T two = ky > 0 ? T(1) : T(0);  // the row -ky, if there is one
    T er = 0, ei = 0, br = 0, bi = 0;    // E+ plus / minus E- parts
    T fr = 0, fi = 0, dr = 0, di = 0;
#pragma unroll 4
    for (int kx = 0; kx <= K; ++kx) {
      const T cs = tw[kx][l][0], sn = tw[kx][l][1];
      const T pr = (T)cp[2 * kx], pi = (T)cp[2 * kx + 1];
      const T mr = two * (T)cm[2 * kx], mi = two * (T)cm[2 * kx + 1];
      const T xr = pr * cs - pi * sn, xi = pr * sn + pi * cs;
      const T yr = mr * cs - mi * sn, yi = mr * sn + mi * cs;
      er += xr;
      ei += xi;
      fr += yr;
      fi += yi;
      br += (T)kx * xr;
      bi += (T)kx * xi;
      dr += (T)kx * yr;
      di += (T)kx * yi;
    }
    T* o = W + (((size_t)s * (K + 1) + ky) * 4) * nx + ix;
    o[0] = -gy * (T)ky * (ei - fi);
    o[nx] = -gy * (T)ky * (er + fr);
    o[2 * (size_t)nx] = gx * (bi + di);
    o[3 * (size_t)nx] = gx * (br - dr);
  }
}

// 2D, pass 2 (along y): a wavefront takes 64 sites of kFlowIy rows, so that
// a loaded W serves kFlowIy rows; the twiddles of the block's rows in LDS.
constexpr int kFlowIy = 8;
template <typename T>
__global__ __launch_bounds__(kFlowBlock) void k_flow2d_y(
    const T* __restrict__ W, int K, int nx, int ny, T* __restrict__ u) {
  constexpr int NW = kFlowBlock / 64, R = NW * kFlowIy;
  __shared__ __align__(16) T tw[65][R][2];
  const int y0 = (int)blockIdx.y * R;
  const int64_t s = blockIdx.z;
  for (int i = (int)threadIdx.x; i < (K + 1) * R; i += kFlowBlock) {
    const int k = i / R, r = i - k * R;
    T cs, sn;
    phase_k<T>((uint32_t)k, (uint32_t)(y0 + r < ny ? y0 + r : 0), (uint32_t)ny,
               &cs, &sn);
    tw[k][r][0] = cs;
    tw[k][r][1] = sn;
  }
  __syncthreads();
  const int l = (int)threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int ix = (int)blockIdx.x * 64 + l;
  if (ix >= nx) return;
  T ux[kFlowIy] = {}, uy[kFlowIy] = {};
  const T* a = W + ((size_t)s * (K + 1) * 4) * nx + ix;
#pragma unroll 2
  for (int k = 0; k <= K; ++k, a += 4 * (size_t)nx) {
    const T w0 = a[0], w1 = a[nx], w2 = a[2 * (size_t)nx],
            w3 = a[3 * (size_t)nx];
#pragma unroll
    for (int r = 0; r < kFlowIy; ++r) {
      const T cs = tw[k][w * kFlowIy + r][0], sn = tw[k][w * kFlowIy + r][1];
      ux[r] += w0 * cs + w1 * sn;
      uy[r] += w2 * cs + w3 * sn;
    }
  }
  const size_t plane = (size_t)nx * ny;
  T* const o = u + (size_t)s * 2 * plane + ix;
#pragma unroll
  for (int r = 0; r < kFlowIy; ++r) {
    const int iy = y0 + w * kFlowIy + r;
    if (iy < ny) {
      o[(size_t)iy * nx] = ux[r];
      o[plane + (size_t)iy * nx] = uy[r];
    }
  }
}

// Bound by launches and latency for a few slices, by the store of u for
// many: 8 slices of 512^2 with K = 32 10.5 and 21 us, where a thread per site
// and row with its own twiddles, and per site of one y, took 26.6 and 146 us.
template <typename T>
hipError_t flow2d(const float* coef, int K, int64_t nx, int64_t ny, double dx,
                  int64_t ns, T* u, T* work, int64_t chunk, hipStream_t st) {
  const T gx = (T)(2.0 * M_PI / ((double)nx * dx));
  const T gy = (T)(2.0 * M_PI / ((double)ny * dx));
  const unsigned bx = (unsigned)((nx + 63) / 64);
  const unsigned bk = (unsigned)((K + kFlowRows) / kFlowRows);
  const int R = kFlowBlock / 64 * kFlowIy;
  const unsigned by = (unsigned)((ny + R - 1) / R);
  for (int64_t s = 0; s < ns; s += chunk) {
    const unsigned n = (unsigned)(ns - s < chunk ? ns - s : chunk);
    hipLaunchKernelGGL(k_flow2d_x<T>, dim3(bx, bk, n), dim3(kFlowBlock), 0, st,
                       coef + (size_t)s * (2 * K + 1) * (K + 1) * 2, K,
                       (int)nx, gx, gy, work);
    hipLaunchKernelGGL(k_flow2d_y<T>, dim3(bx, by, n), dim3(kFlowBlock), 0, st,
                       work, K, (int)nx, (int)ny,
                       u + (size_t)s * 2 * (size_t)(nx * ny));
  }
  return hipGetLastError();
}

// Workspace of flow2d, kept by the handle (at most kFlowWork bytes, or one
// slice's): slices go through it in chunks.  Under stream capture a
// stream-ordered allocation that belongs to the graph is used instead, so
// that a captured call does not depend on the handle's buffer.  The kept one
// is stream-ordered too: hipMalloc is refused, and ends the capture, while
// any other stream of the process is being captured.
constexpr size_t kFlowWork = (size_t)32 << 20;
template <typename T>
hipError_t flow2d_call(lattice_t* L, const float* coef, int K, int64_t ns,
                       T* u) {
  const lattice_desc& d = L->d;
  const size_t slice = sizeof(T) * 4 * (size_t)(K + 1) * (size_t)d.nx;
  int64_t chunk = (int64_t)(kFlowWork / slice);
  chunk = chunk < 1 ? 1 : (chunk > ns ? ns : chunk);
  const size_t need = slice * (size_t)chunk;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipError_t e = hipSuccess;
  if (L->stream)  // the null stream is never captured
    e = hipStreamIsCapturing(L->stream, &cap);
  if (e != hipSuccess) return e;
  if (cap != hipStreamCaptureStatusNone) {
    T* work = nullptr;
    e = hipMallocAsync((void**)&work, need, L->stream);
    if (e != hipSuccess) return e;
    e = flow2d<T>(coef, K, d.nx, d.ny, d.dx, ns, u, work, chunk, L->stream);
    const hipError_t f = hipFreeAsync(work, L->stream);
    return e != hipSuccess ? e : f;
  }
  if (L->flow_bytes < need) {
    if (L->flow_work) (void)hipFreeAsync(L->flow_work, L->stream);
    L->flow_work = nullptr;
    L->flow_bytes = 0;
    e = hipMallocAsync(&L->flow_work, need, L->stream);
    if (e != hipSuccess) {
      L->flow_work = nullptr;
      return e;
    }
    L->flow_bytes = need;
  }
  return flow2d<T>(coef, K, d.nx, d.ny, d.dx, ns, u, (T*)L->flow_work, chunk,
                   L->stream);
}

}  // namespace
}  // namespace lat

extern "C" {

int lattice_flow1d_modes(lattice_t* L, int32_t nmodes, const float* coef,
                         int64_t n_slices, void* u) {
  if (!L) return LATTICE_EINVAL;
  const lattice_desc& d = L->d;
  if (d.dim != 1 || !coef || !u || nmodes < 1 || n_slices < 1 ||
      n_slices > 65535)
    return LATTICE_EINVAL;
  const dim3 grid((unsigned)((d.nx + lat::kFlowBlock - 1) / lat::kFlowBlock),
                  (unsigned)n_slices);
  if (d.dtype == LATTICE_F64)
    hipLaunchKernelGGL(lat::k_flow1d<double>, grid, dim3(lat::kFlowBlock), 0,
                       L->stream, coef, nmodes, (int64_t)d.nx, (double*)u);
  else
    hipLaunchKernelGGL(lat::k_flow1d<float>, grid, dim3(lat::kFlowBlock), 0,
                       L->stream, coef, nmodes, (int64_t)d.nx, (float*)u);
  return hipGetLastError() == hipSuccess ? LATTICE_OK : LATTICE_EHIP;
}

int lattice_flow2d_modes(lattice_t* L, int32_t kmax, const float* coef,
                         int64_t n_slices, void* u) {
  if (!L) return LATTICE_EINVAL;
  const lattice_desc& d = L->d;
  if (d.dim != 2 || !coef || !u || kmax < 1 || kmax > 64 || n_slices < 1 ||
      n_slices > 65535 || d.ny > 65535 || 2 * kmax >= d.nx ||
      2 * kmax >= d.ny)
    return LATTICE_EINVAL;
  const hipError_t e =
      d.dtype == LATTICE_F64
          ? lat::flow2d_call<double>(L, coef, kmax, n_slices, (double*)u)
          : lat::flow2d_call<float>(L, coef, kmax, n_slices, (float*)u);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return LATTICE_EHIP;
  }
  return LATTICE_OK;
}

}  // extern "C"
