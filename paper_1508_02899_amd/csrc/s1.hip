// s1.hip -- Eulerian first-order velocity structure function of the
// phase-space density (Eq. 11, Sec. 3.1), gfx950.
//
//   S1(r) = < sum_{j,j'} f_j(x) f_j'(x + r) |v_j - v_j'| >_x
//           / < sum_{j,j'} f_j(x) f_j'(x + r) >_x.
//
// With h_j(y) = sum_j' |v_j - v_j'| f_j'(y) (velocity units of dv), the
// numerator is < sum_j f_j(x) h_j(x + r) >_x and the denominator
// < rho(x) rho(x + r) >_x (rho = sum_j f_j; every dv factor but the one of
// |v - v'| cancels).  1D: h by a direct sum over j' per site.  2D:
// |v_J - v_J'| = dv |J - J'| (Euclidean on the velocity square), so h is
// the product of the state (sites x nv^2) with the fixed nv^2 x nv^2 matrix
// of index distances -- a plain GEMM, done by rocBLAS.  The correlation
// sums for each requested separation are FP64 with fixed-order reductions.
// In 2D the separation r is taken along x and along y and the two
// estimates are averaged.
#include <math.h>

#include <rocblas/rocblas.h>

#include <type_traits>

#include "../../include/lattice.h"
#include "device_common.h"
#include "lattice_internal.h"
#include "lattice_struct.h"

namespace lat {
namespace {

constexpr int kS1Block = 256;

// 1D: h[j][x] = sum_j' |j - j'| f[j'][x]
template <typename T>
__global__ __launch_bounds__(kS1Block) void k_s1_h1d(const T* __restrict__ f,
                                                     int64_t nx, int nv,
                                                     T* __restrict__ h) {
  const int64_t x = (int64_t)blockIdx.x * kS1Block + threadIdx.x;
  const int j = blockIdx.y;
  if (x >= nx) return;
  T acc = 0;
  for (int jp = 0; jp < nv; ++jp)
    acc += (T)(jp > j ? jp - j : j - jp) * f[(size_t)jp * nx + x];
  h[(size_t)j * nx + x] = acc;
}

// 2D distance matrix D[J'][J] = |J - J'| on the nv x nv index square
template <typename T>
__global__ __launch_bounds__(kS1Block) void k_s1_dist(int nv, T* __restrict__ D) {
  const int64_t n2 = (int64_t)nv * nv;
  const int64_t i = (int64_t)blockIdx.x * kS1Block + threadIdx.x;
  if (i >= n2 * n2) return;
  const int64_t a = i / n2, b = i - a * n2;
  const int ay = (int)(a / nv), ax = (int)(a - ay * nv);
  const int by = (int)(b / nv), bx = (int)(b - by * nv);
  const double dxv = ax - bx, dyv = ay - by;
  D[i] = (T)sqrt(dxv * dxv + dyv * dyv);
}

constexpr int kS1Sites = 2;  // sites per thread of k_s1_num

// A set of up to NQ separations: along x (dx sites, already mod nx) or along
// y (dy, mod ny), one of the two being zero.
template <int NQ>
struct S1Seps {
  int32_t dx[NQ], dy[NQ];
};

// Partial sums of sum_J f_J(x) h_J(x') over a chunk of sites and a group of
// planes, for NQ separations at once: f is read once for all of them and the
// shifted h's come from the caches (the workgroups of an XCD work on the
// same few planes, xcd_remap).  Bound by the h loads: 12 separations of
// 256^2 x 17^2 take 71 us, where a pass per separation that also summed
// rho(x) and rho(x') took 197 us.
// partial[q nblocks + block].
template <typename T, int NQ>
__global__ __launch_bounds__(kS1Block) void k_s1_num(
    const T* __restrict__ f, int64_t fpitch, const T* __restrict__ h, int nx,
    int ny, int nplanes, int nchunks, int per, S1Seps<NQ> sep,
    double* __restrict__ partial) {
  __shared__ double sh[NQ][kS1Block / 64];
  const int sites = nx * ny;
  const int blk = xcd_remap((int)blockIdx.x, (int)gridDim.x);
  const int grp = blk / nchunks, chunk = blk - grp * nchunks;
  const int J0 = grp * per, J1 = min(J0 + per, nplanes);
  int at[kS1Sites], to[kS1Sites][NQ];
  bool in[kS1Sites];
#pragma unroll
  for (int e = 0; e < kS1Sites; ++e) {
    const int64_t i = ((int64_t)chunk * kS1Sites + e) * kS1Block + threadIdx.x;
    in[e] = i < sites;
    at[e] = in[e] ? (int)i : 0;
    const int y = at[e] / nx, x = at[e] - y * nx;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      // unsigned: both below 2^31, so the sums stay below 2^32
      uint32_t xs = (uint32_t)x + (uint32_t)sep.dx[q];
      uint32_t ys = (uint32_t)y + (uint32_t)sep.dy[q];
      if (xs >= (uint32_t)nx) xs -= (uint32_t)nx;
      if (ys >= (uint32_t)ny) ys -= (uint32_t)ny;
      to[e][q] = (int)(ys * (uint32_t)nx + xs);
    }
  }
  double acc[NQ] = {};
  for (int J = J0; J < J1; ++J) {
    const T* const fj = f + (size_t)J * fpitch;
    const T* const hj = h + (size_t)J * sites;
    T a[kS1Sites], b[kS1Sites][NQ];
#pragma unroll
    for (int e = 0; e < kS1Sites; ++e) {
      a[e] = fj[at[e]];
#pragma unroll
      for (int q = 0; q < NQ; ++q) b[e][q] = hj[to[e][q]];
    }
#pragma unroll
    for (int e = 0; e < kS1Sites; ++e) {
      const double d = in[e] ? (double)a[e] : 0.0;
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (in[e]) acc[q] += d * (double)b[e][q];
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc[q] += __shfl_xor(acc[q], o);
    if (((int)threadIdx.x & 63) == 0) sh[q][threadIdx.x >> 6] = acc[q];
  }
  __syncthreads();
  if ((int)threadIdx.x < NQ) {
    const double* p = sh[threadIdx.x];
    partial[(size_t)threadIdx.x * gridDim.x + blk] =
        (p[0] + p[1]) + (p[2] + p[3]);
  }
}

__device__ double block_sum(double a, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  if (((int)threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Partial sums of rho(x) rho(x') over a chunk of sites of one separation.
constexpr int kDenSites = 4;  // sites per thread
template <int NQ>
__global__ __launch_bounds__(kS1Block) void k_s1_den(
    const double* __restrict__ rho, int nx, int ny, S1Seps<NQ> sep,
    double* __restrict__ partial) {
  __shared__ double sh[kS1Block / 64];
  const int64_t sites = (int64_t)nx * ny;
  const int q = blockIdx.y;
  double acc = 0.0;
#pragma unroll 4
  for (int e = 0; e < kDenSites; ++e) {
    const int64_t i =
        ((int64_t)blockIdx.x * kDenSites + e) * kS1Block + threadIdx.x;
    if (i < sites) {
      const int y = (int)(i / nx), x = (int)(i - (int64_t)y * nx);
      uint32_t xs = (uint32_t)x + (uint32_t)sep.dx[q];
      uint32_t ys = (uint32_t)y + (uint32_t)sep.dy[q];
      if (xs >= (uint32_t)nx) xs -= (uint32_t)nx;
      if (ys >= (uint32_t)ny) ys -= (uint32_t)ny;
      acc += rho[i] * rho[(size_t)ys * nx + xs];
    }
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) partial[(size_t)q * gridDim.x + blockIdx.x] = acc;
}

// out[2 q], out[2 q + 1]: fixed-order sums of separation q's partials.
__global__ __launch_bounds__(kS1Block) void k_s1_final(
    const double* __restrict__ num, int nnum, const double* __restrict__ den,
    int nden, double* __restrict__ out) {
  __shared__ double sh[2][kS1Block / 64];
  const int q = blockIdx.x;
  double a = 0.0, b = 0.0;
  for (int j = threadIdx.x; j < nnum; j += kS1Block)
    a += num[(size_t)q * nnum + j];
  for (int j = threadIdx.x; j < nden; j += kS1Block)
    b += den[(size_t)q * nden + j];
  a = block_sum(a, sh[0]);
  b = block_sum(b, sh[1]);
  if (threadIdx.x == 0) {
    out[2 * q] = a;
    out[2 * q + 1] = b;
  }
}

// Workgroups of k_s1_num: chunks of sites, times groups of `per` planes so
// that a few thousand workgroups run whatever the sizes are.
struct S1Grid {
  int nchunks, per, groups;
  int64_t nden;  // workgroups per separation of k_s1_den
};

S1Grid s1_grid(int64_t sites, int nplanes) {
  S1Grid g;
  g.nchunks = (int)((sites + kS1Block * kS1Sites - 1) / (kS1Block * kS1Sites));
  int groups = (2048 + g.nchunks - 1) / g.nchunks;
  groups = groups < 1 ? 1 : (groups > nplanes ? nplanes : groups);
  g.per = (nplanes + groups - 1) / groups;
  g.groups = (nplanes + g.per - 1) / g.per;
  g.nden = (sites + kS1Block * kDenSites - 1) / (kS1Block * kDenSites);
  return g;
}

// Separations first .. first + nq - 1 (in the order r[0] along x, r[0] along
// y, r[1] along x, ...) into sums[2 q], q < nq; nq <= NQ.
template <typename T, int NQ>
hipError_t correlate(const T* f, int64_t fpitch, const T* h,
                     const double* rho, int64_t nx, int64_t ny, int nplanes,
                     const int32_t* r, int naxes, int first, int nq,
                     const S1Grid& g, double* partial, double* sums,
                     hipStream_t st) {
  S1Seps<NQ> sep = {};
  for (int q = 0; q < nq; ++q) {
    const int k = (first + q) / naxes, axis = (first + q) - k * naxes;
    if (axis == 0)
      sep.dx[q] = (int32_t)(r[k] % nx);
    else
      sep.dy[q] = (int32_t)(r[k] % ny);
  }
  const int nb = g.nchunks * g.groups;
  double* const den = partial + (size_t)NQ * nb;
  hipLaunchKernelGGL((k_s1_num<T, NQ>), dim3(nb), dim3(kS1Block), 0, st, f,
                     fpitch, h, (int)nx, (int)ny, nplanes, g.nchunks, g.per,
                     sep, partial);
  hipLaunchKernelGGL((k_s1_den<NQ>), dim3((unsigned)g.nden, nq),
                     dim3(kS1Block), 0, st, rho, (int)nx, (int)ny, sep, den);
  hipLaunchKernelGGL(k_s1_final, dim3(nq), dim3(kS1Block), 0, st, partial, nb,
                     den, (int)g.nden, sums + 2 * first);
  return hipGetLastError();
}

constexpr int kS1MaxQ = 16;

template <typename T>
hipError_t correlate_all(const T* f, int64_t fpitch, const T* h,
                         const double* rho, int64_t nx, int64_t ny,
                         int nplanes, const int32_t* r, int naxes, int total,
                         const S1Grid& g, double* partial, double* sums,
                         hipStream_t st) {
  for (int first = 0; first < total; first += kS1MaxQ) {
    const int nq = total - first < kS1MaxQ ? total - first : kS1MaxQ;
    auto go = [&](auto n) {
      return correlate<T, decltype(n)::value>(f, fpitch, h, rho, nx, ny,
                                              nplanes, r, naxes, first, nq, g,
                                              partial, sums, st);
    };
    // unused slots of a set load h like the used ones: the smallest set
    const hipError_t e =
        nq <= 4 ? go(std::integral_constant<int, 4>())
        : nq <= 8 ? go(std::integral_constant<int, 8>())
        : nq <= 12 ? go(std::integral_constant<int, 12>())
                   : go(std::integral_constant<int, kS1MaxQ>());
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace
}  // namespace lat

extern "C" int lattice_s1(lattice_t* L, const void* f, double dt, int32_t nr,
                          const int32_t* r, double* out) {
  if (!L) return LATTICE_EINVAL;
  const lattice_desc& d = L->d;
  if (!f || !r || !out || nr < 1 || nr > 4096 || !(dt > 0.0) ||
      !isfinite(dt))
    return LATTICE_EINVAL;
  for (int k = 0; k < nr; ++k)
    if (r[k] < 0) return LATTICE_EINVAL;
  const bool f64 = d.dtype == LATTICE_F64;
  const size_t el = f64 ? 8 : 4;
  const int64_t sites = L->sites;
  const int naxes = d.dim == 2 ? 2 : 1;
  const int64_t np = L->nplanes;
  const int total = nr * naxes;
  hipStream_t st = L->stream;
  // workspace: rho, the partial sums of one set of separations, the sums
  const lat::S1Grid g = lat::s1_grid(sites, (int)np);
  const size_t npart =
      (size_t)lat::kS1MaxQ * ((size_t)g.nchunks * g.groups + (size_t)g.nden);
  const size_t need = sizeof(double) * ((size_t)sites + npart +
                                        2 * (size_t)total);
  if (L->s1_bytes < need) {
    if (L->s1_work) (void)hipFree(L->s1_work);
    L->s1_work = nullptr;
    L->s1_bytes = 0;
    if (hipMalloc((void**)&L->s1_work, need) != hipSuccess) {
      L->s1_work = nullptr;
      return LATTICE_ENOMEM;
    }
    L->s1_bytes = need;
  }
  double* const rho = L->s1_work;
  double* const partial = rho + sites;
  double* const sums = partial + npart;
  void* const h = L->scratch;  // at least the cells of a state
  int rc = LATTICE_OK;
  hipError_t e = hipSuccess;
  if (d.dim == 1) {
    const dim3 gh((unsigned)((d.nx + lat::kS1Block - 1) / lat::kS1Block),
                  (unsigned)d.nv);
    if (f64)
      hipLaunchKernelGGL(lat::k_s1_h1d<double>, gh, dim3(lat::kS1Block), 0, st,
                         (const double*)f, (int64_t)d.nx, d.nv, (double*)h);
    else
      hipLaunchKernelGGL(lat::k_s1_h1d<float>, gh, dim3(lat::kS1Block), 0, st,
                         (const float*)f, (int64_t)d.nx, d.nv, (float*)h);
    e = hipGetLastError();
  } else {
    const size_t nD = (size_t)np * np;
    if (!L->s1_dist) {
      if (hipMalloc(&L->s1_dist, el * nD) != hipSuccess) {
        L->s1_dist = nullptr;
        return LATTICE_ENOMEM;
      }
      const unsigned gd = (unsigned)((nD + lat::kS1Block - 1) / lat::kS1Block);
      if (f64)
        hipLaunchKernelGGL(lat::k_s1_dist<double>, dim3(gd),
                           dim3(lat::kS1Block), 0, st, d.nv,
                           (double*)L->s1_dist);
      else
        hipLaunchKernelGGL(lat::k_s1_dist<float>, dim3(gd),
                           dim3(lat::kS1Block), 0, st, d.nv,
                           (float*)L->s1_dist);
      e = hipGetLastError();
      if (e != hipSuccess) {  // not filled: the next call starts over
        (void)hipFree(L->s1_dist);
        L->s1_dist = nullptr;
        return LATTICE_EHIP;
      }
    }
    rocblas_handle handle = (rocblas_handle)L->s1_blas;
    if (!handle) {
      if (rocblas_create_handle(&handle) != rocblas_status_success)
        return LATTICE_EHIP;
      if (rocblas_set_stream(handle, st) != rocblas_status_success) {
        rocblas_destroy_handle(handle);
        return LATTICE_EHIP;
      }
      L->s1_blas = handle;
    }
    // column-major view: F (sites x np, ld = the plane pitch), D (np x np),
    // h = F D (sites x np, ld sites)
    rocblas_status bs;
    if (f64) {
      const double one = 1.0, zero = 0.0;
      bs = rocblas_dgemm(handle, rocblas_operation_none,
                         rocblas_operation_none, (rocblas_int)sites,
                         (rocblas_int)np, (rocblas_int)np, &one,
                         (const double*)f, (rocblas_int)L->pitch,
                         (const double*)L->s1_dist, (rocblas_int)np, &zero,
                         (double*)h, (rocblas_int)sites);
    } else {
      const float one = 1.f, zero = 0.f;
      bs = rocblas_sgemm(handle, rocblas_operation_none,
                         rocblas_operation_none, (rocblas_int)sites,
                         (rocblas_int)np, (rocblas_int)np, &one,
                         (const float*)f, (rocblas_int)L->pitch,
                         (const float*)L->s1_dist, (rocblas_int)np, &zero,
                         (float*)h, (rocblas_int)sites);
    }
    if (bs != rocblas_status_success) rc = LATTICE_EHIP;
  }
  if (rc == LATTICE_OK && e == hipSuccess)
    e = lat::launch_density(f, sites, L->pitch, (int)np, f64, 1.0, rho, st);
  if (rc == LATTICE_OK && e == hipSuccess) {
    const int64_t ny = d.dim == 2 ? d.ny : 1;
    e = f64 ? lat::correlate_all((const double*)f, L->pitch, (const double*)h,
                                 rho, d.nx, ny, (int)np, r, naxes, total, g,
                                 partial, sums, st)
            : lat::correlate_all((const float*)f, L->pitch, (const float*)h,
                                 rho, d.nx, ny, (int)np, r, naxes, total, g,
                                 partial, sums, st);
  }
  // pinned memory for the usual few separations
  double* hs = 2 * total <= lat::kHostRed ? L->host_red
                                          : new (std::nothrow) double[2 * total];
  if (!hs) rc = LATTICE_ENOMEM;
  if (rc == LATTICE_OK && e == hipSuccess)
    e = hipMemcpyAsync(hs, sums, sizeof(double) * 2 * total,
                       hipMemcpyDeviceToHost, st);
  const hipError_t es = hipStreamSynchronize(st);
  if (e == hipSuccess) e = es;
  if (e != hipSuccess) {
    (void)hipGetLastError();
    rc = LATTICE_EHIP;
  }
  if (rc == LATTICE_OK) {
    const double dv = (double)d.vstride * d.dx / dt;
    for (int k = 0; k < nr; ++k) {
      double s = 0.0;
      for (int a = 0; a < naxes; ++a) {
        const double* q = hs + 2 * ((size_t)k * naxes + a);
        s += dv * q[0] / q[1];
      }
      out[k] = s / naxes;
      if (!isfinite(out[k])) rc = LATTICE_ENONFINITE;
    }
  }
  if (hs != L->host_red) delete[] hs;
  return rc;
}

namespace lat {
void s1_release(lattice_t* L) {
  if (L->s1_blas) rocblas_destroy_handle((rocblas_handle)L->s1_blas);
  if (L->s1_dist) (void)hipFree(L->s1_dist);
  if (L->s1_work) (void)hipFree(L->s1_work);
}
}  // namespace lat
