// Gamma-index evaluation (the dose agreement test of Sec. 3.1, after Low et
// al. 1998): gamma(r) = min over r' of sqrt((D_ref(r) - D_eval(r'))^2 / dD^2 +
// |r - r'|^2 / dr^2), with r' on a lattice of step dr / substeps around the
// voxel centre r and D_eval trilinearly interpolated between voxel centres
// (clamped at the grid's outer centres).
//
// One lane per reference voxel.  The search lattice is cut into the cells of
// eight voxel centres that its points fall into (GammaCell, the same around
// every voxel, ascending in their smallest distance; wave-uniform, read
// through the scalar path).  A lane is finished once the distance alone
// reaches its best value, the loop ends when every lane is.  Per cell a lane
// loads the eight doses once and forms the trilinear polynomial; a lane whose
// dose lies outside their range by more than its best value allows skips the
// cell, and a cell that all lanes skip costs only the loads.  Its points then
// take three multiply-adds each, with the weights uniform; a point at a time,
// eight gathers and the weights per lane each, took 57 FP64 operations
// (256x256x160, 2 %/2 mm, 5 substeps, 3.5e6 voxels of mean gamma 0.29: 6.8 ms,
// now 1.18 ms).  Bound by the latency of the cells' loads and by lanes that wait
// for the slower ones of their wave.
//
// All arithmetic is FP64 in units of one lattice step: best is gamma^2 s^2
// (s = substeps), distances are whole numbers, doses are scaled by s / dD.
// The pass decision gamma < 1 is best < s^2.
#include <hip/hip_runtime.h>

#include "ctd_internal.h"

namespace ctd {

namespace {

// A cell's points: lattice offsets i in [i0, i1), j in [j0, j1), k in
// [k0, k1) (indices into the weight tables), those with i^2 + j^2 + k^2 <= r2max.
// BORDER: some lane's cell leaves the grid; there the interpolation is that
// at the clamped coordinate: the outermost cell with weight 0 or 1.
template <bool BORDER>
__device__ __forceinline__ double cell_min(const GammaTables &t, const GammaCell &c,
                                           const double e[8], double dr, double best,
                                           const bool lo[3], const bool hi[3]) {
  // A + fz B with A, B bilinear in (fx, fy)
  const double c0 = e[0], cx = e[1] - e[0], cy = e[2] - e[0], cxy = (e[3] - e[2]) - cx;
  const double d0 = e[4] - e[0], dx = (e[5] - e[4]) - cx, dy = (e[6] - e[4]) - cy,
               dxy = ((e[7] - e[6]) - (e[5] - e[4])) - cxy;
  for (int j = c.j0; j < c.j1; ++j) {
    double fy = t.fy[j];
    if (BORDER) fy = lo[1] ? 0.0 : hi[1] ? 1.0 : fy;
    const int y = j - t.L, y2 = y * y;
    for (int i = c.i0; i < c.i1; ++i) {
      double fx = t.fx[i];
      if (BORDER) fx = lo[0] ? 0.0 : hi[0] ? 1.0 : fx;
      const int x = i - t.L, r2 = x * x + y2;
      if (!__any((double)r2 < best)) continue;   // (lanes in this cell)
      const double A = dr - fma(fy, fma(fx, cxy, cy), fma(fx, cx, c0));
      const double B = fma(fy, fma(fx, dxy, dy), fma(fx, dx, d0));
      double m = INFINITY;
      for (int k = c.k0; k < c.k1; ++k) {
        const int z = k - t.L;
        if (r2 + z * z > t.r2max) continue;
        double fz = t.fz[k];
        if (BORDER) fz = lo[2] ? 0.0 : hi[2] ? 1.0 : fz;
        const double d = fma(-fz, B, A);
        m = fmin(m, fma(d, d, (double)(z * z)));
      }
      best = fmin(best, m + (double)r2);
    }
  }
  return best;
}

// Cell index of a voxel index and a cell's offset, which for voxels far smaller
// than a lattice step lies at the end of the int range: saturating (one
// instruction), so that such a cell stays beyond the grid's edge.
__device__ __forceinline__ int cell_at(int i, int offset) {
  return __builtin_elementwise_add_sat(i, offset);
}

// The eight doses of the cell with lower corner j: at its border the outermost
// cell's, with lo / hi the axes whose weight is clamped to 0 / 1.
template <bool BORDER>
__device__ __forceinline__ void load_cell(const float *__restrict__ ev, int nx, int ny, int nz,
                                          const int j[3], float f[8], bool lo[3], bool hi[3]) {
  const int64_t sy = nx, sz = (int64_t)nx * ny;
  if constexpr (BORDER) {
    const int nn[3] = {nx, ny, nz};
    int a0[3], a1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = j[a] < 0 || nn[a] == 1;
      hi[a] = j[a] > nn[a] - 2;
      a0[a] = max(min(j[a], nn[a] - 2), 0);
      a1[a] = min(a0[a] + 1, nn[a] - 1);
    }
    const float *p00 = ev + a0[2] * sz + a0[1] * sy, *p01 = ev + a0[2] * sz + a1[1] * sy;
    const float *p10 = ev + a1[2] * sz + a0[1] * sy, *p11 = ev + a1[2] * sz + a1[1] * sy;
    f[0] = p00[a0[0]]; f[1] = p00[a1[0]]; f[2] = p01[a0[0]]; f[3] = p01[a1[0]];
    f[4] = p10[a0[0]]; f[5] = p10[a1[0]]; f[6] = p11[a0[0]]; f[7] = p11[a1[0]];
  } else {
    const float *p = ev + ((int64_t)j[2] * sz + (int64_t)j[1] * sy + j[0]);
    f[0] = p[0]; f[1] = p[1]; f[2] = p[sy]; f[3] = p[sy + 1];
    f[4] = p[sz]; f[5] = p[sz + 1]; f[6] = p[sz + sy]; f[7] = p[sz + sy + 1];
  }
}

// Whether the dose at the centre of voxel (ix, iy, iz) counts: the interpolant
// there is formed from the eight doses of the voxel's cell, and is not a number
// where one of them is not finite.
__device__ __forceinline__ bool centre_finite(const float *__restrict__ ev, int nx, int ny, int nz,
                                              int ix, int iy, int iz) {
  const int j[3] = {ix, iy, iz};
  float f[8];
  bool lo[3], hi[3];
  load_cell<true>(ev, nx, ny, nz, j, f, lo, hi);
  uint32_t top = 0u;
#pragma unroll
  for (int a = 0; a < 8; ++a) top = max(top, __float_as_uint(f[a]) & 0x7FFFFFFFu);
  return top < 0x7F800000u;
}

// best over the cell of lattice points around voxel (ix, iy, iz), or `best`
// where the eight doses rule the cell out.
template <bool BORDER>
__device__ __forceinline__ double visit(const GammaTables &t, const GammaCell &c,
                                        const float *__restrict__ ev, int nx, int ny, int nz,
                                        int ix, int iy, int iz, double dr, double best,
                                        double scale) {
  const int j[3] = {cell_at(ix, c.cx), cell_at(iy, c.cy), cell_at(iz, c.cz)};
  float f[8];
  bool lo[3], hi[3];
  load_cell<BORDER>(ev, nx, ny, nz, j, f, lo, hi);
  const float fl = fminf(fminf(fminf(f[0], f[1]), fminf(f[2], f[3])),
                         fminf(fminf(f[4], f[5]), fminf(f[6], f[7])));
  const float fh = fmaxf(fmaxf(fmaxf(f[0], f[1]), fmaxf(f[2], f[3])),
                         fmaxf(fmaxf(f[4], f[5]), fmaxf(f[6], f[7])));
  // the interpolant stays within [fl, fh] up to a few roundings, which the
  // margin covers
  const double gap = fmax(fmax((double)fl * scale - dr, dr - (double)fh * scale), 0.0);
  if (fma(gap, gap, (double)c.r2min) * (1.0 - 0x1p-40) >= best) return best;
  double e[8];
#pragma unroll
  for (int a = 0; a < 8; ++a) e[a] = (double)f[a] * scale;
  return cell_min<BORDER>(t, c, e, dr, best, lo, hi);
}

__device__ __forceinline__ double lane_f64(double v, int lane) {
  const uint64_t b = __double_as_longlong(v);
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readlane((uint32_t)b, lane);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
  return __longlong_as_double((long long)(hi << 32 | lo));
}

}  // namespace

// With at most kFewLanes lanes of a wave still searching, the wave turns to
// one of their voxels at a time, a cell per lane: a voxel without a near match
// walks hundreds of cells, which its wave would otherwise wait for one by one
// (65 K voxels, 2 %/3 mm: 680 us without, 175 us with it; at 4 / 8 / 16 / 24
// lanes the head grid takes 6.1 / 5.4 / 5.7 / 6.3 ms a call at 5 % noise).
constexpr int kFewLanes = 8;

// gamma may be null; counts (kGammaSlots pairs, one 128-byte line each) the
// voxels with D_ref > region and those with gamma < 1.
__global__ void __launch_bounds__(256) k_gamma(const float *__restrict__ ref,
                                               const float *__restrict__ ev, int nx, int ny,
                                               int nz, GammaTables t,
                                               double scale, double region, double cap2,
                                               float *__restrict__ gamma,
                                               unsigned long long *__restrict__ counts) {
  __shared__ unsigned int n_region, n_pass;
  if (threadIdx.x == 0) n_region = n_pass = 0u;
  __syncthreads();
  const int64_t V = (int64_t)nx * ny * nz;
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool active = false;
  double dr = 0.0, best = cap2;
  int ix = 0, iy = 0, iz = 0;
  if (v < V) {
    const double r = (double)ref[v];
    active = r > region;
    dr = r * scale;
    ix = (int)(v % nx);
    const int64_t row = v / nx;
    iy = (int)(row % ny);
    iz = (int)(row / ny);
  }
  if (active && centre_finite(ev, nx, ny, nz, ix, iy, iz)) {   // it bounds the search
    const double d = dr - (double)ev[v] * scale;
    best = fmin(best, d * d);
  }
  int q = 0;
  for (; q < t.n_cells; ++q) {
    const GammaCell &c = t.cells[q];
    const bool want = active && (double)c.r2min < best;
    const int left = __popcll(__ballot(want));
    if (left <= kFewLanes) break;   // none included
    const int jx = cell_at(ix, c.cx), jy = cell_at(iy, c.cy), jz = cell_at(iz, c.cz);
    const bool in = (unsigned)jx < (unsigned)(nx - 1) && (unsigned)jy < (unsigned)(ny - 1) &&
                    (unsigned)jz < (unsigned)(nz - 1);
    if (__all(in || !want)) {
      if (want) best = visit<false>(t, c, ev, nx, ny, nz, ix, iy, iz, dr, best, scale);
    } else if (want) {
      best = visit<true>(t, c, ev, nx, ny, nz, ix, iy, iz, dr, best, scale);
    }
  }
  if (q < t.n_cells) {
    const int lane = threadIdx.x & 63;
    unsigned long long m = __ballot(active && (double)t.cells[q].r2min < best);
    for (; m; m &= m - 1) {
      const int j = __builtin_ctzll(m);
      const int vx = __builtin_amdgcn_readlane(ix, j), vy = __builtin_amdgcn_readlane(iy, j),
                vz = __builtin_amdgcn_readlane(iz, j);
      const double vdr = lane_f64(dr, j);
      double b = lane_f64(best, j);
      for (int q0 = q; q0 < t.n_cells; q0 += 64) {
        const GammaCell &c = t.cells[min(q0 + lane, t.n_cells - 1)];
        const bool want = q0 + lane < t.n_cells && (double)c.r2min < b;
        if (!__any(want)) break;   // cells ascend in r2min
        double mine = b;
        if (want) mine = visit<true>(t, c, ev, nx, ny, nz, vx, vy, vz, vdr, b, scale);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mine = fmin(mine, __shfl_xor(mine, o, 64));
        b = mine;
      }
      if (lane == j) best = b;
    }
  }
  const double s2 = (double)t.s2;
  if (gamma && v < V) gamma[v] = active ? (float)sqrt(best / s2) : -1.0f;
  const unsigned long long m_reg = __ballot(active), m_pass = __ballot(active && best < s2);
  if ((threadIdx.x & 63) == 0 && m_reg) {
    atomicAdd(&n_region, (unsigned)__popcll(m_reg));
    atomicAdd(&n_pass, (unsigned)__popcll(m_pass));
  }
  __syncthreads();
  if (threadIdx.x == 0 && n_region) {
    unsigned long long *o = counts + 16 * (blockIdx.x % kGammaSlots);
    atomicAdd(&o[0], (unsigned long long)n_region);
    if (n_pass) atomicAdd(&o[1], (unsigned long long)n_pass);
  }
}

int launch_gamma(const float *ref, const float *ev, int nx, int ny, int nz, const GammaTables &t,
                 double scale, double region, double cap2, float *gamma,
                 unsigned long long *counts, void *stream) {
  const int64_t V = (int64_t)nx * ny * nz;
  if (V <= 0) return 0;
  const int64_t blocks = (V + 255) / 256;
  if (blocks > 0x7fffffff) return -1;
  hipLaunchKernelGGL(k_gamma, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, ref, ev,
                     nx, ny, nz, t, scale, region, cap2, gamma, counts);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ctd
