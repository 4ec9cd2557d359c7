// observables.hip -- coarse-grained density statistics (gfx950).
//
// rho_r on non-overlapping tilings with boxes of r = 2^k lattice spacings
// per direction (the paper's coarse-grained density of Sec. 3.2, tiled
// rather than sliding): the box mass m_b is the sum of the site densities
// inside, rho_r = (m_b / M) * N_b so that <rho_r> = 1, and
//   <rho_r^2> = N_b * sum_b m_b^2 / M^2.
// Level k + 1 box masses are the sums of 2^dim level-k boxes.  All sums are
// FP64 in a fixed order.
//
// Bound by launches and latency, not by bytes (a density is 0.1 to 2 MB): a
// workgroup takes a tile of 32 x 32 sites (1024 in 1D) through all the levels
// inside it (6; 11 in 1D), a second stage does the same on the tiles' masses,
// and a last stage of one workgroup also combines the levels.  8 levels at
// 128^2: 2 launches, 11 us; a launch per level: 9 launches, 39 us.
#include "device_common.h"
#include "lattice_internal.h"

namespace lat {
namespace {

constexpr int kObsBlock = 256;
constexpr int kMaxLevels = kRhoMaxLevels;
constexpr int kTile = 1024;  // sites per workgroup: 32 x 32, or 1024 in 1D

// Levels that one tile holds: boxes of 1 .. 32 (1 .. 1024) sites per side.
constexpr int stage_levels(int dim) { return dim == 2 ? 6 : 11; }

struct LevelMeta {
  int64_t off[kMaxLevels], nblk[kMaxLevels], nbox[kMaxLevels];
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// out[k] = N_b * sum m^2 / (sum m)^2 from level k's partial sums; levels
// q, q + 4, ... by wavefront q.
__device__ void combine_levels(const double* partial, const LevelMeta& meta,
                               int levels, double* out) {
  const int l = (int)threadIdx.x & 63;
  for (int k = (int)threadIdx.x >> 6; k < levels; k += kObsBlock / 64) {
    const double* p = partial + 2 * meta.off[k];
    double s1 = 0.0, s2 = 0.0;
    for (int64_t j = l; j < meta.nblk[k]; j += 64) {
      s1 += p[2 * j];
      s2 += p[2 * j + 1];
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (l == 0) out[k] = (double)meta.nbox[k] * s2 / (s1 * s1);
  }
}

// One stage: the box masses m_in[ny][nx] of level `base` (the sites when
// base = 0) are summed over the boxes of levels base .. base + nlev - 1.
// Sums of m and m^2 of level k over this tile go to partial[2 (off[k] +
// tile)]; level `base` itself only in the first stage (the stage before has
// done it).  Boxes lie wholly inside or outside the array (nx and ny are
// multiples of the largest box), so cells outside count as zeros.  m_out
// (when not NULL) gets the mass of the whole tile.
template <int DIM>
__global__ __launch_bounds__(kObsBlock) void k_tile_stage(
    const double* __restrict__ m_in, int64_t nx, int64_t ny, int64_t ntx,
    int base, int nlev, LevelMeta meta, double* partial,
    double* __restrict__ m_out, int levels, double* __restrict__ out) {
  constexpr int NL = stage_levels(DIM);
  __shared__ double box[kObsBlock], red[NL][kObsBlock / 64][2];
  const int t = (int)threadIdx.x, l = t & 63, w = t >> 6;
  const int64_t tile = blockIdx.x;
  double v[4];  // 2 x 2 sites (2D) or 4 consecutive ones (1D)
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    int64_t x, y;
    if (DIM == 2) {
      const int64_t ty = tile / ntx, tx = tile - ty * ntx;
      x = tx * 32 + 2 * (t & 15) + (e & 1);
      y = ty * 32 + 2 * (t >> 4) + (e >> 1);
    } else {
      x = tile * kTile + 4 * t + e;
      y = 0;
    }
    v[e] = x < nx && y < ny ? m_in[y * nx + x] : 0.0;
  }
  auto note = [&](int k, double s1, double s2) {
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (l == 0) {
      red[k][w][0] = s1;
      red[k][w][1] = s2;
    }
  };
  note(0, (v[0] + v[1]) + (v[2] + v[3]),
       (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]));
  const double a = v[0] + v[1], b = v[2] + v[3];
  double m = a + b;
  int k = 1;
  if (DIM == 1) {
    note(1, m, a * a + b * b);
    k = 2;
  }
  note(k, m, m * m);
  // the remaining levels halve the number of boxes (per side)
  int side = DIM == 2 ? 16 : kObsBlock;  // boxes (per side) of level k
  for (++k; k < nlev; ++k) {
    __syncthreads();
    if (t < (DIM == 2 ? side * side : side)) box[t] = m;
    __syncthreads();
    const int half = side / 2;
    const bool in = t < (DIM == 2 ? half * half : half);
    m = 0.0;
    if (in && DIM == 2) {
      const double* r = box + (2 * (t / half)) * side + 2 * (t % half);
      m = (r[0] + r[1]) + (r[side] + r[side + 1]);
    } else if (in) {
      m = box[2 * t] + box[2 * t + 1];
    }
    side = half;
    note(k, m, m * m);
  }
  if (t == 0 && m_out) m_out[tile] = m;
  __syncthreads();
  if (t < nlev && (t > 0 || base == 0)) {
    double s1 = red[t][0][0], s2 = red[t][0][1];
#pragma unroll
    for (int q = 1; q < kObsBlock / 64; ++q) {
      s1 += red[t][q][0];
      s2 += red[t][q][1];
    }
    double* p = partial + 2 * (meta.off[base + t] + tile);
    p[0] = s1;
    p[1] = s2;
  }
  if (out) {  // the last stage, one workgroup
    __threadfence_block();
    __syncthreads();
    combine_levels(partial, meta, levels, out);
  }
}

__global__ __launch_bounds__(kObsBlock) void k_tile_combine(
    const double* __restrict__ partial, LevelMeta meta, int levels,
    double* __restrict__ out) {
  combine_levels(partial, meta, levels, out);
}

struct Stage {
  int64_t nx, ny, ntx, tiles;  // input boxes, tiles
};

Stage stage_of(int dim, int64_t nx, int64_t ny) {
  const int64_t ntx = dim == 2 ? (nx + 31) / 32 : (nx + kTile - 1) / kTile;
  return {nx, ny, ntx, dim == 2 ? ntx * ((ny + 31) / 32) : ntx};
}

}  // namespace

int64_t rho_r2_work(int dim, int64_t nx, int64_t ny) {
  // every level's partials (a pair per tile of its stage), the tile masses
  // of every stage, the results
  int64_t n = kMaxLevels;
  Stage st = stage_of(dim, nx, dim == 2 ? ny : 1);
  for (int base = 0; base < kMaxLevels; base += stage_levels(dim) - 1) {
    n += (2 * stage_levels(dim) + 1) * st.tiles;
    st = stage_of(dim, st.ntx, st.tiles / st.ntx);
  }
  return n;
}

hipError_t launch_rho_r2(const double* rho, int dim, int64_t nx, int64_t ny,
                         int levels, double* work, hipStream_t s) {
  LevelMeta meta = {};
  double* const out = work;
  const double* in = rho;
  const int NL = stage_levels(dim);
  // sizes of the stages, then their launches
  Stage st[kMaxLevels];
  int nst = 0;
  int64_t poff = 0, n = nx * (dim == 2 ? ny : 1);
  for (int base = 0; base < levels; base += NL - 1) {
    if (base > 0 && base == levels - 1) break;  // done by the stage before
    const Stage* p = nst ? &st[nst - 1] : nullptr;
    st[nst] = p ? stage_of(dim, p->ntx, p->tiles / p->ntx)
                : stage_of(dim, nx, dim == 2 ? ny : 1);
    for (int k = base ? base + 1 : 0; k < levels && k < base + NL; ++k) {
      meta.off[k] = poff;
      meta.nblk[k] = st[nst].tiles;
      meta.nbox[k] = n >> (dim * k);
      poff += st[nst].tiles;
    }
    ++nst;
  }
  double* const partial = work + kMaxLevels;
  double* masses = partial + 2 * poff;
  bool combined = false;
  for (int i = 0; i < nst; ++i) {
    const int base = i * (NL - 1);
    const int nlev = levels - base < NL ? levels - base : NL;
    const bool last = i == nst - 1;
    double* const mo = last ? nullptr : masses;
    combined = last && st[i].tiles == 1;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)st[i].tiles),
                         dim3(kObsBlock), 0, s, in, st[i].nx, st[i].ny,
                         st[i].ntx, base, nlev, meta, partial, mo, levels,
                         combined ? out : nullptr);
    };
    if (dim == 2)
      go(k_tile_stage<2>);
    else
      go(k_tile_stage<1>);
    in = mo;
    masses += st[i].tiles;
  }
  if (!combined)
    hipLaunchKernelGGL(k_tile_combine, dim3(1), dim3(kObsBlock), 0, s, partial,
                       meta, levels, out);
  return hipGetLastError();
}

}  // namespace lat
