// aux_kernels.hip -- FP64 conservation moments, density, flow checks and
// copies for the lattice library (gfx950).
#include <float.h>

#include "device_common.h"
#include "lattice_internal.h"

namespace lat {
namespace {

constexpr int kBlock = 256;

// Fixed-order block reduction of one double per thread: a pairwise tree in
// LDS, the same pairing on every run, so results are bit-reproducible.
__device__ double block_sum(double v, double* sh) {
  const int t = (int)threadIdx.x;
  sh[t] = v;
  __syncthreads();
#pragma unroll
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if (t < w) sh[t] = sh[t] + sh[t + w];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// One workgroup per velocity plane: sum of the plane's sites in FP64.
// When the plane is 16-byte aligned and a whole number of 16-byte pieces,
// thread t adds pieces t, t+256, ... (coalesced 16-byte loads, one FP64
// partial sum per element of a piece, combined in a fixed order);
// otherwise sites t, t+256, ... one by one.  Then the tree.  The order of
// the additions depends only on the plane size, so repeated calls give the
// same bits.
template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
  typedef float4 type;
  static constexpr int n = 4;
};
template <>
struct Vec16<double> {
  typedef double2 type;
  static constexpr int n = 2;
};

template <typename T>
__global__ __launch_bounds__(kBlock) void k_plane_sums(const T* __restrict__ f,
                                                       int64_t sites,
                                                       int64_t pitch,
                                                       double* __restrict__ out) {
  __shared__ double sh[kBlock];
  using V = typename Vec16<T>::type;
  constexpr int NE = Vec16<T>::n;
  const T* p = f + (size_t)blockIdx.x * (size_t)pitch;
  double acc = 0.0;
  if (sites % NE == 0 && ((uintptr_t)p & 15) == 0) {  // uniform
    const V* q = reinterpret_cast<const V*>(p);
    const int64_t n = sites / NE;
    double a[NE] = {};
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < n; i += kBlock) {
      const V v = q[i];
      const T* e = reinterpret_cast<const T*>(&v);
#pragma unroll
      for (int k = 0; k < NE; ++k) a[k] += (double)e[k];
    }
#pragma unroll
    for (int k = 0; k < NE; ++k) acc += a[k];
  } else {
    for (int64_t i = threadIdx.x; i < sites; i += kBlock) acc += (double)p[i];
  }
  const double s = block_sum(acc, sh);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// Weighted combination of the plane sums: M = w sum S_j, P_k = w sum S_j v_k,
// Q_k = w sum S_j v_k^2 with v = (j - h) dv per component, and the variance
// sum_k Q_k/M - |P/M|^2.  Single workgroup, fixed order: lanes and then
// wavefronts by a tree.  Latency-bound: the five sums go through one tree
// together (4225 planes: 5.5 us; 9.3 us with 256 threads and a tree per sum).
constexpr int kMomWaves = 16;
__global__ __launch_bounds__(64 * kMomWaves) void k_moments_final(
    const double* __restrict__ ps, int nv, int dim, double w, double dv,
    const int* __restrict__ flag, double* __restrict__ out) {
  __shared__ double sh[kMomWaves][5];
  const int h = (nv - 1) / 2;
  const int nplanes = dim == 1 ? nv : nv * nv;
  double a[5] = {};  // m, px, py, qx, qy
#pragma unroll 4
  for (int j = threadIdx.x; j < nplanes; j += 64 * kMomWaves) {
    const double s = ps[j];
    const int jy = dim == 2 ? j / nv : 0;
    const double vx = (double)(j - jy * nv - h) * dv;
    const double vy = dim == 2 ? (double)(jy - h) * dv : 0.0;
    a[0] += s;
    a[1] += s * vx;
    a[3] += s * vx * vx;
    a[2] += s * vy;
    a[4] += s * vy * vy;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int k = 0; k < 5; ++k) a[k] += __shfl_xor(a[k], o);
  const int l = (int)threadIdx.x & 63, q = (int)threadIdx.x >> 6;
  if (l == 0)
#pragma unroll
    for (int k = 0; k < 5; ++k) sh[q][k] = a[k];
  __syncthreads();
  if (q != 0) return;
#pragma unroll
  for (int k = 0; k < 5; ++k) a[k] = sh[l % kMomWaves][k];
#pragma unroll
  for (int o = kMomWaves / 2; o > 0; o >>= 1)
#pragma unroll
    for (int k = 0; k < 5; ++k) a[k] += __shfl_xor(a[k], o);
  if (l == 0) {
    const double m = a[0], px = a[1], py = a[2], qx = a[3], qy = a[4];
    out[0] = w * m;
    out[1] = w * px;
    out[2] = w * py;
    out[3] = w * qx;
    out[4] = w * qy;
    const double var = (qx + qy) / m - ((px / m) * (px / m) + (py / m) * (py / m));
    out[5] = var;
    out[6] = (double)*flag;
  }
}

// rho[site] = dvd * sum_j f[j][site] in FP64.  Bound by the one read of the
// state; a lane per site walking all the planes leaves too few loads in
// flight when the sites are few and the planes many.  Here NW wavefronts
// share 64 VEC consecutive sites: wavefront w adds planes w, w + NW, ...
// (eight loads in flight), and the NW sums are added in wavefront order.
// The order of the additions depends only on the sizes.  Measured against a
// lane per site: 128^2 x 65^2 1422 -> 41 us (6.7 TB/s), 512^2 x 33^2 492 ->
// 212 us (5.4 TB/s), 192^2 x 17^2 FP64 70 -> 14 us.
template <typename T, int VEC>
struct alignas(sizeof(T) * VEC) SiteVec {
  T v[VEC];
};

template <typename T, int VEC, int NW>
__global__ __launch_bounds__(64 * NW) void k_density(
    const T* __restrict__ f, int64_t sites, int64_t pitch, int nplanes,
    double dvd, double* __restrict__ rho) {
  using V = SiteVec<T, VEC>;
  __shared__ double sh[NW][64 * VEC];
  const int l = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
  const int64_t s0 = (int64_t)blockIdx.x * (64 * VEC);
  const int64_t i = s0 + l * VEC;
  double a[VEC] = {};
  if (i < sites) {  // VEC divides sites
    const T* p = f + i;
    int j = w;
    for (; j + 7 * NW < nplanes; j += 8 * NW) {
      V v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        v[k] = *(const V*)(p + (size_t)(j + k * NW) * pitch);
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int e = 0; e < VEC; ++e) a[e] += (double)v[k].v[e];
    }
    for (; j < nplanes; j += NW) {
      const V v = *(const V*)(p + (size_t)j * pitch);
#pragma unroll
      for (int e = 0; e < VEC; ++e) a[e] += (double)v.v[e];
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) sh[w][l * VEC + e] = a[e];
  __syncthreads();
  for (int t = (int)threadIdx.x; t < 64 * VEC; t += 64 * NW) {
    if (s0 + t >= sites) break;
    double r = sh[0][t];
#pragma unroll
    for (int q = 1; q < NW; ++q) r += sh[q][t];
    rho[s0 + t] = dvd * r;
  }
}

// A lane per site, walking all the planes, U loads in flight.
template <typename T, int U>
__global__ __launch_bounds__(kBlock) void k_density_lane(
    const T* __restrict__ f, int64_t sites, int64_t pitch, int nplanes,
    double dvd, double* __restrict__ rho) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= sites) return;
  const T* p = f + i;
  double acc = 0.0;
#pragma unroll U
  for (int j = 0; j < nplanes; ++j, p += pitch) acc += (double)*p;
  rho[i] = dvd * acc;
}

// Many sites fill the chip with a lane per site, and there the wavefronts of
// a workgroup that read several planes at once gain nothing (us, FP32 unless
// said; "wide" is 16-byte loads by 4 or 16 wavefronts):
//   sites that no 16-byte load divides: 1048577 x 3, 17, 65, 81 planes 6.2,
//   19.3, 87.8, 120.7 by 4 or 16 wavefronts, 4.4, 14.5, 50.2, 73.2 by a lane
//   with two loads in flight; 262145 x 289, 1089 62.7, 240, 80, 323 with two
//   loads and 50.9, 193 with eight;
//   planes that all start on the same memory channels (a multiple of 64 KiB
//   apart): 524288 x 33, 65 planes wide 18.4, 36.3, two wavefronts with
//   4-byte loads 11.7, 21.1, but 1048576 x 9 9.4, 11.4; FP64 262144 x 33, 65,
//   81 wide 17.8, 36.5, 37.9, a lane 11.8, 20.8, 25.3, 524288 x 9, 289 8.4, 230,
//   7.3, 203, but 262144 x 17 5.5, 7.4 and 4194304 x 33 196, 207;
//   elsewhere 800000 x 33, 65 wide 18.3, 31.7, two wavefronts 16.9, 32.3.
template <typename T>
void density_go(const T* f, int64_t sites, int64_t pitch, int nplanes,
                double dvd, double* rho, hipStream_t s) {
  constexpr int VEC = 16 / (int)sizeof(T);
  const bool aligned = sites % VEC == 0 && pitch % VEC == 0 &&
                       ((uintptr_t)f & 15) == 0;
  // 16-byte loads once they still leave two workgroups per compute unit,
  // and only where every plane and the sites allow the alignment
  const bool wide = sites >= (int64_t)64 * VEC * 512 && aligned;
  auto go = [&](auto kernel, int per, int threads) {
    const int64_t g = (sites + per - 1) / per;
    hipLaunchKernelGGL(kernel, dim3((unsigned)g), dim3(threads), 0, s, f,
                       sites, pitch, nplanes, dvd, rho);
  };
  if (sites >= 262144 && !aligned)
    return nplanes < 96 ? go(k_density_lane<T, 2>, kBlock, kBlock)
                        : go(k_density_lane<T, 8>, kBlock, kBlock);
  if (sites >= 262144 && (uint64_t)pitch * sizeof(T) % 65536 == 0) {
    if (sizeof(T) == 4 && nplanes >= 17 && nplanes < 128)
      return go(k_density<T, 1, 2>, 64, 128);
    if (sizeof(T) == 8 && sites <= (1 << 21) &&
        (sites >= 524288 || (nplanes >= 32 && nplanes < 128)))
      return go(k_density_lane<T, 1>, kBlock, kBlock);
  }
  // 16 wavefronts where each still has a run of planes to add
  if (nplanes >= 64) {
    if (wide)
      go(k_density<T, VEC, 16>, 64 * VEC, 64 * 16);
    else
      go(k_density<T, 1, 16>, 64, 64 * 16);
  } else {
    if (wide)
      go(k_density<T, VEC, 4>, 64 * VEC, 64 * 4);
    else
      go(k_density<T, 1, 4>, 64, 64 * 4);
  }
}

// Flow check: flag |= 1 if some |u| exceeds umax_ok (>= when strict) or is
// not finite.  Grid-stride, one atomic per offending wavefront.
// With n16 > 0 also the copy of n16 16-byte pieces and tail more bytes that a
// call of an odd number of passes starts with: one launch instead of two,
// which is what a call of a single step on a small lattice consists of.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_cfl_check(
    const T* __restrict__ u, int64_t n, T umax_ok, int strict,
    int* __restrict__ flag, const uint4* __restrict__ src,
    uint4* __restrict__ dst, int64_t n16, int tail) {
  bool bad = false;
  if (blockIdx.x == 0 && (int)threadIdx.x < tail)
    ((char*)(dst + n16))[threadIdx.x] =
        ((const char*)(src + n16))[threadIdx.x];
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n16;
       i += stride)
    dst[i] = src[i];
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += stride) {
    const T a = u[i] < T(0) ? -u[i] : u[i];
    const bool ok = strict ? (a < umax_ok) : (a <= umax_ok);  // NaN -> !ok
    bad |= !ok;
  }
  if (__any(bad) && ((int)threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

// max |u| into out (out must hold 0 beforehand); NaN propagates as +inf.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_absmax(const T* __restrict__ u,
                                                   int64_t n,
                                                   unsigned long long* out) {
  __shared__ double sh[kBlock];
  double m = 0.0;
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += stride) {
    double a = (double)u[i];
    a = a < 0 ? -a : a;
    if (!(a <= DBL_MAX)) a = __longlong_as_double(0x7ff0000000000000LL);
    m = a > m ? a : m;
  }
  const int t = (int)threadIdx.x;
  sh[t] = m;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if (t < w) sh[t] = sh[t] > sh[t + w] ? sh[t] : sh[t + w];
    __syncthreads();
  }
  // non-negative doubles order like their bit patterns
  if (t == 0) atomicMax(out, (unsigned long long)__double_as_longlong(sh[0]));
}

__global__ __launch_bounds__(kBlock) void k_copy16(const uint4* __restrict__ s,
                                                   uint4* __restrict__ d,
                                                   int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += stride)
    d[i] = s[i];
}

__global__ void k_copy1(const unsigned char* __restrict__ s,
                        unsigned char* __restrict__ d, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) d[i] = s[i];
}

__global__ void k_clear(int* flag) { *flag = 0; }

__global__ void k_flag_out(const int* flag, int32_t* status) {
  *status = *flag;
}

__global__ void k_clear_u64(unsigned long long* p) { *p = 0ull; }

int grid_for(int64_t n) {
  int64_t g = (n + kBlock - 1) / kBlock;
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  return (int)g;
}

}  // namespace

hipError_t launch_moments(const void* f, int64_t sites, int64_t pitch,
                          int nv, int dim, int f64, double w, double dv,
                          double* plane_sums, const int* flag, double* out,
                          hipStream_t s) {
  const int nplanes = dim == 1 ? nv : nv * nv;
  if (f64)
    hipLaunchKernelGGL(k_plane_sums<double>, dim3(nplanes), dim3(kBlock), 0, s,
                       (const double*)f, sites, pitch, plane_sums);
  else
    hipLaunchKernelGGL(k_plane_sums<float>, dim3(nplanes), dim3(kBlock), 0, s,
                       (const float*)f, sites, pitch, plane_sums);
  hipLaunchKernelGGL(k_moments_final, dim3(1), dim3(64 * kMomWaves), 0, s,
                     plane_sums, nv, dim, w, dv, flag, out);
  return hipGetLastError();
}

hipError_t launch_density(const void* f, int64_t sites, int64_t pitch,
                          int nplanes, int f64, double dvd, double* rho,
                          hipStream_t s) {
  if (f64)
    density_go((const double*)f, sites, pitch, nplanes, dvd, rho, s);
  else
    density_go((const float*)f, sites, pitch, nplanes, dvd, rho, s);
  return hipGetLastError();
}

hipError_t launch_check_copy(const void* u, int64_t n, double umax_ok,
                             int strict, int f64, int* flag, void* dst,
                             const void* src, int64_t bytes, hipStream_t s) {
  const bool whole = ((uintptr_t)dst % 16) == 0 && ((uintptr_t)src % 16) == 0;
  if (!whole) {  // misaligned copies by themselves
    const hipError_t e = launch_copy(dst, src, bytes, s);
    if (e != hipSuccess) return e;
  }
  const int64_t n16 = whole ? bytes / 16 : 0;
  const int tail = whole ? (int)(bytes % 16) : 0;
  const int g = grid_for(n > n16 ? n : n16);
  if (f64)
    hipLaunchKernelGGL(k_cfl_check<double>, dim3(g), dim3(kBlock), 0, s,
                       (const double*)u, n, umax_ok, strict, flag,
                       (const uint4*)src, (uint4*)dst, n16, tail);
  else
    hipLaunchKernelGGL(k_cfl_check<float>, dim3(g), dim3(kBlock), 0, s,
                       (const float*)u, n, (float)umax_ok, strict, flag,
                       (const uint4*)src, (uint4*)dst, n16, tail);
  return hipGetLastError();
}

hipError_t launch_absmax(const void* u, int64_t n, int f64, double* out,
                         hipStream_t s) {
  auto* o = reinterpret_cast<unsigned long long*>(out);
  hipLaunchKernelGGL(k_clear_u64, dim3(1), dim3(1), 0, s, o);
  const int g = grid_for(n);
  if (f64)
    hipLaunchKernelGGL(k_absmax<double>, dim3(g), dim3(kBlock), 0, s,
                       (const double*)u, n, o);
  else
    hipLaunchKernelGGL(k_absmax<float>, dim3(g), dim3(kBlock), 0, s,
                       (const float*)u, n, o);
  return hipGetLastError();
}

hipError_t launch_copy(void* dst, const void* src, int64_t bytes,
                       hipStream_t s) {
  const int64_t n16 = bytes / 16;
  if (n16 > 0 && ((uintptr_t)dst % 16) == 0 && ((uintptr_t)src % 16) == 0) {
    hipLaunchKernelGGL(k_copy16, dim3(grid_for(n16)), dim3(kBlock), 0, s,
                       (const uint4*)src, (uint4*)dst, n16);
    const int64_t done = n16 * 16;
    const int64_t rest = bytes - done;
    if (rest > 0)
      hipLaunchKernelGGL(k_copy1, dim3(1), dim3(64), 0, s,
                         (const unsigned char*)src + done,
                         (unsigned char*)dst + done, rest);
  } else if (bytes > 0) {
    hipLaunchKernelGGL(k_copy1, dim3((int)((bytes + 255) / 256)), dim3(256), 0,
                       s, (const unsigned char*)src, (unsigned char*)dst,
                       bytes);
  }
  return hipGetLastError();
}

hipError_t launch_clear_flag(int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_clear, dim3(1), dim3(1), 0, s, flag);
  return hipGetLastError();
}

hipError_t launch_flag_out(const int* flag, int32_t* status, hipStream_t s) {
  hipLaunchKernelGGL(k_flag_out, dim3(1), dim3(1), 0, s, flag, status);
  return hipGetLastError();
}

}  // namespace lat
