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

// The separations of one launch, r mod nx (mod ny where they are along y):
// with naxes = 2, even ones along x and odd ones along y.  Few of them travel
// as kernel arguments, more in device memory (at; zeros past the last one).  A
// launch takes them in sets of NQ, set blockIdx.y: a launch per set made many
// separations of a short lattice a matter of launches (4096 x 17, 40 of them:
// one launch for all 42 us, one per 16 86, one for all again 37; 600 of
// them 72, 565, 75).
constexpr int kS1Few = 48;
struct S1Seps {
  const int32_t* at;
  int32_t r[kS1Few];
  __device__ __forceinline__ uint32_t get(int g) const {
    return (uint32_t)(at ? at[g] : r[g]);
  }
};

// Partial sums of sum_J f_J(x) h_J(x') over a chunk of sites and a group of
// planes, for NQ separations at once: f is read once for all of them and the
// shifted h's come from the caches (the workgroups of an XCD work on the
// same few planes, xcd_remap).  Bound by the h loads: 12 separations of
// 256^2 x 17^2 take 71 us, where a pass per separation that also summed
// rho(x) and rho(x') took 197 us.
// partial[(set NQ + q) nblocks + block].
template <typename T, int NQ>
__global__ __launch_bounds__(kS1Block) void k_s1_num(
    const T* __restrict__ f, int64_t fpitch, const T* __restrict__ h, int nx,
    int ny, int nplanes, int nchunks, int per, S1Seps sep,
    int naxes, double* __restrict__ partial) {
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
      const int g = (int)blockIdx.y * NQ + q;
      const uint32_t r = sep.get(g);
      const bool along_y = naxes == 2 && (g & 1);
      uint32_t xs = (uint32_t)x + (along_y ? 0u : r);
      uint32_t ys = (uint32_t)y + (along_y ? r : 0u);
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
    partial[((size_t)blockIdx.y * NQ + threadIdx.x) * gridDim.x + blk] =
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
__global__ __launch_bounds__(kS1Block) void k_s1_den(
    const double* __restrict__ rho, int nx, int ny, S1Seps sep, int naxes,
    double* __restrict__ partial) {
  __shared__ double sh[kS1Block / 64];
  const int64_t sites = (int64_t)nx * ny;
  const int q = blockIdx.y;
  const bool along_y = naxes == 2 && (q & 1);
  const uint32_t r = sep.get(q);
  const uint32_t dx = along_y ? 0u : r, dy = along_y ? r : 0u;
  double acc = 0.0;
#pragma unroll 4
  for (int e = 0; e < kDenSites; ++e) {
    const int64_t i =
        ((int64_t)blockIdx.x * kDenSites + e) * kS1Block + threadIdx.x;
    if (i < sites) {
      const int y = (int)(i / nx), x = (int)(i - (int64_t)y * nx);
      uint32_t xs = (uint32_t)x + dx;
      uint32_t ys = (uint32_t)y + dy;
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

// How `total` separations are cut into sets of nq (4, 8, 12 or 16, the fewest
// loads: an f per set and an h per slot, the unused ones included), and the
// workgroups of k_s1_num: chunks of sites, times groups of `per` planes so
// that a few thousand run in all sets together, whatever the sizes are (the
// order of a separation's additions depends on the sizes and on `total`).
struct S1Cut {
  int nq, sets;  // sets of a launch: the partial sums stay below 16 MB
  int nchunks, per, groups;
  int64_t nden;  // workgroups per separation of k_s1_den
  size_t npart;  // doubles of partial sums
};

S1Cut s1_cut(int total, int64_t sites, int nplanes) {
  S1Cut c = {};
  int64_t best = -1;
  for (int nq = 16; nq >= 4; nq -= 4) {
    const int64_t cost = (int64_t)((total + nq - 1) / nq) * (nq + 2);
    if (best < 0 || cost < best) {
      best = cost;
      c.nq = nq;
    }
  }
  c.sets = (total + c.nq - 1) / c.nq;
  c.nchunks = (int)((sites + kS1Block * kS1Sites - 1) / (kS1Block * kS1Sites));
  const int64_t blocks = (int64_t)c.nchunks * c.sets;
  int64_t groups = (2048 + blocks - 1) / blocks;
  groups = groups < 1 ? 1 : (groups > nplanes ? nplanes : groups);
  c.per = (int)((nplanes + groups - 1) / groups);
  c.groups = (nplanes + c.per - 1) / c.per;
  c.nden = (sites + kS1Block * kDenSites - 1) / (kS1Block * kDenSites);
  const size_t set =
      (size_t)c.nq * ((size_t)c.nchunks * c.groups + (size_t)c.nden);
  while (c.sets > 1 && (size_t)c.sets * set > ((size_t)1 << 21))
    c.sets = (c.sets + 1) / 2;
  c.npart = (size_t)c.sets * set;
  return c;
}

// Separations first .. first + n - 1 (r[0] along x, r[0] along y, r[1] along
// x, ..., each modulo the lattice; first is a multiple of 4) into
// sums[2 first ..].
template <typename T, int NQ>
hipError_t correlate(const T* f, int64_t fpitch, const T* h,
                     const double* rho, int64_t nx, int64_t ny, int nplanes,
                     const S1Seps& seps, int naxes, int first, int n,
                     const S1Cut& c, double* partial, double* sums,
                     hipStream_t st) {
  S1Seps sep = seps;
  if (sep.at) sep.at += first;
  const int nb = c.nchunks * c.groups;
  const int sets = (n + NQ - 1) / NQ;
  double* const den = partial + (size_t)sets * NQ * nb;
  hipLaunchKernelGGL((k_s1_num<T, NQ>), dim3(nb, sets), dim3(kS1Block), 0, st,
                     f, fpitch, h, (int)nx, (int)ny, nplanes, c.nchunks, c.per,
                     sep, naxes, partial);
  hipLaunchKernelGGL(k_s1_den, dim3((unsigned)c.nden, n), dim3(kS1Block), 0,
                     st, rho, (int)nx, (int)ny, sep, naxes, den);
  hipLaunchKernelGGL(k_s1_final, dim3(n), dim3(kS1Block), 0, st, partial, nb,
                     den, (int)c.nden, sums + 2 * first);
  return hipGetLastError();
}

template <typename T>
hipError_t correlate_all(const T* f, int64_t fpitch, const T* h,
                         const double* rho, int64_t nx, int64_t ny,
                         int nplanes, const S1Seps& seps, int naxes, int total,
                         const S1Cut& c, double* partial, double* sums,
                         hipStream_t st) {
  const int most = c.sets * c.nq;
  for (int first = 0; first < total; first += most) {
    const int n = total - first < most ? total - first : most;
    auto go = [&](auto nq) {
      return correlate<T, decltype(nq)::value>(f, fpitch, h, rho, nx, ny,
                                               nplanes, seps, naxes, first, n,
                                               c, partial, sums, st);
    };
    const hipError_t e =
        c.nq == 4 ? go(std::integral_constant<int, 4>())
        : c.nq == 8 ? go(std::integral_constant<int, 8>())
        : c.nq == 12 ? go(std::integral_constant<int, 12>())
                     : go(std::integral_constant<int, 16>());
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
  // workspace: rho, the partial sums of one launch's separations, the sums,
  // the separations (when they do not go as kernel arguments)
  const lat::S1Cut cut = lat::s1_cut(total, sites, (int)np);
  const int slots = (total + cut.nq - 1) / cut.nq * cut.nq;
  const bool few = slots <= lat::kS1Few;
  const size_t need = sizeof(double) * ((size_t)sites + cut.npart +
                                        2 * (size_t)total) +
                      sizeof(int32_t) * (few ? 0 : (size_t)slots);
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
  double* const sums = partial + cut.npart;
  int32_t* const at = few ? nullptr : (int32_t*)(sums + 2 * (size_t)total);
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
  lat::S1Seps seps = {at, {}};
  int32_t* const rs = few ? seps.r : new (std::nothrow) int32_t[slots];
  if (!rs) rc = LATTICE_ENOMEM;
  for (int q = 0; rs && q < slots; ++q)
    rs[q] = q >= total ? 0
                       : (int32_t)(r[q / naxes] %
                                   (q % naxes == 0 ? d.nx : d.ny));
  if (rc == LATTICE_OK && e == hipSuccess && !few)
    e = hipMemcpyAsync(at, rs, sizeof(int32_t) * slots, hipMemcpyHostToDevice,
                       st);
  if (rc == LATTICE_OK && e == hipSuccess)
    e = lat::launch_density(f, sites, L->pitch, (int)np, f64, 1.0, rho, st);
  if (rc == LATTICE_OK && e == hipSuccess) {
    const int64_t ny = d.dim == 2 ? d.ny : 1;
    e = f64 ? lat::correlate_all((const double*)f, L->pitch, (const double*)h,
                                 rho, d.nx, ny, (int)np, seps, naxes, total,
                                 cut, partial, sums, st)
            : lat::correlate_all((const float*)f, L->pitch, (const float*)h,
                                 rho, d.nx, ny, (int)np, seps, naxes, total,
                                 cut, partial, sums, st);
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
  if (!few) delete[] rs;
  return rc;
}

namespace lat {
void s1_release(lattice_t* L) {
  if (L->s1_blas) rocblas_destroy_handle((rocblas_handle)L->s1_blas);
  if (L->s1_dist) (void)hipFree(L->s1_dist);
  if (L->s1_work) (void)hipFree(L->s1_work);
}
}  // namespace lat
