// Dose comparison tools behind the C ABI: the gamma-index agreement test of
// Sec. 3.1 (kernel in ctd_gamma.hip).
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

#include "ctd.h"
#include "ctd_api_internal.h"

using namespace ctd;

namespace {

constexpr int kMaxOffsets = 1 << 22;
constexpr size_t kToolMaxBytes = (size_t)256 << 20;   // largest block kept between calls

struct Dev {
  void *p = nullptr;
  ~Dev() {
    if (p) (void)hipFree(p);
  }
};

// The lattice offsets of one axis, o = i h / d voxels for i in [-L, L]: the
// cell each falls into, its weight there, and the runs of equal cells.
//
// A cell takes at most kRunMax steps per axis: small cells bound the search
// earlier and give the lanes of a wave even pieces (2 / 3 / 4 / unbounded: 123 /
// 165 / 218 / 522 us for 65 K voxels of 0.4 cm at 0.2 cm, where unbounded cells
// hold up to 125 points; no difference at 0.1 cm, whose cells hold two or three
// steps anyway).
constexpr int kRunMax = 2;
struct Axis {
  std::vector<double> f;
  struct Run {
    int cell, i0, i1, near2;   // near2: smallest (i - L)^2 of the run
  };
  std::vector<Run> runs;
};

Axis gamma_axis(int L, double h, double d) {
  Axis a;
  for (int i = -L; i <= L; ++i) {
    const double o = i * h / d, c = std::floor(o);
    a.f.push_back(o - c);
    // (a lattice beyond the int range of cells lies beyond every grid: its
    // cells clamp to the same outermost one)
    const int cell = (int)std::min(std::max(c, -2147483000.0), 2147483000.0);
    if (a.runs.empty() || a.runs.back().cell != cell ||
        a.runs.back().i1 - a.runs.back().i0 == kRunMax)
      a.runs.push_back({cell, i + L, i + L, i * i});
    a.runs.back().i1 = i + L + 1;
    a.runs.back().near2 = std::min(a.runs.back().near2, i * i);
  }
  return a;
}

// Offsets within the sphere; at most kMaxOffsets + 1 are counted.
int64_t count_offsets(int L, double rmax) {
  int64_t n = 0;
  for (int k = -L; k <= L; ++k)
    for (int j = -L; j <= L; ++j) {
      const double rest = rmax * rmax - (double)(k * k + j * j);
      if (rest < 0) continue;
      int i = (int)std::sqrt(rest);
      while ((double)(i * i) > rest) --i;
      while ((double)((i + 1) * (i + 1)) <= rest) ++i;
      n += 2 * std::min(i, L) + 1;
    }
  return n;
}

}  // namespace

extern "C" int32_t ctd_gamma(ctd_ctx *ctx, const ctd_grid *g, const float *ref, const float *ev,
                             int32_t mem, const ctd_gamma_params *p, float *gamma,
                             uint64_t *n_region, uint64_t *n_pass) {
  if (!ctx) return CTD_EINVAL;
  if (!g || !ref || !ev || !p) return set_err(ctx, CTD_EINVAL, "null argument");
  if (mem != CTD_MEM_HOST && mem != CTD_MEM_DEVICE)
    return set_err(ctx, CTD_EINVAL, "mem must be HOST or DEVICE");
  if (g->nx < 1 || g->ny < 1 || g->nz < 1 || !(g->dx > 0) || !(g->dy > 0) || !(g->dz > 0) ||
      !std::isfinite(g->dx) || !std::isfinite(g->dy) || !std::isfinite(g->dz))
    return set_err(ctx, CTD_EINVAL, "bad grid");
  if (!(p->dose_tol > 0) || !std::isfinite(p->dose_tol) || !(p->dta_cm > 0) ||
      !std::isfinite(p->dta_cm) || !std::isfinite(p->region_min))
    return set_err(ctx, CTD_EINVAL, "dose_tol and dta_cm must be > 0, region_min finite");
  if (!(p->gamma_cap >= 1.0 && p->gamma_cap <= 4.0) || p->substeps < 1 || p->substeps > 20)
    return set_err(ctx, CTD_EINVAL, "need 1 <= gamma_cap <= 4 and 1 <= substeps <= 20");
  const double rmax = p->gamma_cap * p->substeps;   // radius in lattice steps
  const int L = (int)std::ceil(rmax);
  const int64_t offsets = count_offsets(L, rmax);
  if (offsets > kMaxOffsets)
    return set_err(ctx, CTD_EINVAL, "%lld search offsets exceed %d", (long long)offsets,
                   kMaxOffsets);
  const double h = p->dta_cm / p->substeps;
  const Axis ax = gamma_axis(L, h, g->dx), ay = gamma_axis(L, h, g->dy),
             az = gamma_axis(L, h, g->dz);
  GammaTables t{};
  t.L = L;
  t.s2 = p->substeps * p->substeps;
  t.r2max = (int32_t)std::floor(rmax * rmax);
  std::vector<GammaCell> cells;
  for (const Axis::Run &z : az.runs)
    for (const Axis::Run &y : ay.runs)
      for (const Axis::Run &x : ax.runs) {
        const int r2 = x.near2 + y.near2 + z.near2;
        if (r2 > t.r2max) continue;
        cells.push_back(GammaCell{x.cell, y.cell, z.cell, r2, x.i0, x.i1, y.i0, y.i1, z.i0, z.i1,
                                  {0, 0}});
      }
  std::stable_sort(cells.begin(), cells.end(),
                   [](const GammaCell &a, const GammaCell &b) { return a.r2min < b.r2min; });
  t.n_cells = (int32_t)cells.size();
  const int64_t V = (int64_t)g->nx * g->ny * g->nz;
  const hipStream_t st = ctx->stream;
  if (hipSetDevice(ctx->device) != hipSuccess) return set_err(ctx, CTD_EDEVICE, "hipSetDevice");
  // one device block: counters, weights, cells, and (host arrays) both doses
  // and gamma
  const size_t cnt_bytes = kGammaSlots * 16 * sizeof(unsigned long long);
  const size_t w_bytes = 3 * (size_t)(2 * L + 1) * sizeof(double);
  const size_t cell_off = (cnt_bytes + w_bytes + 255) & ~(size_t)255;
  const size_t dose_off = (cell_off + cells.size() * sizeof(GammaCell) + 255) & ~(size_t)255;
  const size_t dose_bytes = ((size_t)V * 4 + 255) & ~(size_t)255;
  const bool to_host = mem == CTD_MEM_HOST && gamma;
  const size_t bytes =
      dose_off + (mem == CTD_MEM_HOST ? (to_host ? 3 : 2) * dose_bytes : (size_t)0);
  Dev d;   // a block too large to keep
  hipError_t e;
  if (bytes > kToolMaxBytes) {
    if ((e = dev_alloc(ctx, &d.p, bytes)) != hipSuccess) return hip_err(ctx, e, "gamma alloc");
  } else if (ctx->tool_cap < bytes) {   // nothing uses it: every call ends with a wait
    if (ctx->tool_ws) (void)hipFree(ctx->tool_ws);
    ctx->tool_ws = nullptr;
    ctx->tool_cap = 0;
    if ((e = dev_alloc(ctx, &ctx->tool_ws, bytes)) != hipSuccess)
      return hip_err(ctx, e, "gamma alloc");
    ctx->tool_cap = bytes;
  }
  char *base = (char *)(d.p ? d.p : ctx->tool_ws);
  unsigned long long *counts = (unsigned long long *)base;
  std::vector<char> tables(dose_off - cnt_bytes);
  double *w = (double *)tables.data();
  std::copy(ax.f.begin(), ax.f.end(), w);
  std::copy(ay.f.begin(), ay.f.end(), w + (2 * L + 1));
  std::copy(az.f.begin(), az.f.end(), w + 2 * (2 * L + 1));
  std::memcpy(tables.data() + (cell_off - cnt_bytes), cells.data(),
              cells.size() * sizeof(GammaCell));
  t.fx = (const double *)(base + cnt_bytes);
  t.fy = t.fx + (2 * L + 1);
  t.fz = t.fy + (2 * L + 1);
  t.cells = (const GammaCell *)(base + cell_off);
  const float *r = ref, *v = ev;
  if (mem == CTD_MEM_HOST) {
    r = (const float *)(base + dose_off);
    v = (const float *)(base + dose_off + dose_bytes);
    if ((e = hipMemcpyAsync((void *)r, ref, 4 * V, hipMemcpyHostToDevice, st)) != hipSuccess ||
        (e = hipMemcpyAsync((void *)v, ev, 4 * V, hipMemcpyHostToDevice, st)) != hipSuccess)
      return hip_err(ctx, e, "gamma upload");
  }
  if ((e = hipMemcpyAsync(base + cnt_bytes, tables.data(), tables.size(), hipMemcpyHostToDevice,
                          st)) != hipSuccess)
    return hip_err(ctx, e, "gamma upload");
  if (launch_zero(counts, cnt_bytes, st) != 0)
    return hip_err(ctx, hipGetLastError(), "gamma launch");
  float *out = to_host ? (float *)(base + dose_off + 2 * dose_bytes) : gamma;
  if (launch_gamma(r, v, g->nx, g->ny, g->nz, t, p->substeps / p->dose_tol, p->region_min,
                   rmax * rmax, out, counts, st) != 0)
    return hip_err(ctx, hipGetLastError(), "gamma launch");
  if (to_host) {
    void *dst = gamma;
    const int rc = read_planes(ctx, V, 1, 4, &dst, [&](int64_t v0, int n, void *slot) {
      return hipMemcpyAsync(slot, out + v0, 4 * (size_t)n, hipMemcpyDeviceToHost, st) ==
                     hipSuccess ? 0 : -1;
    });
    if (rc != CTD_OK) return rc;
  }
  std::vector<unsigned long long> cnt(cnt_bytes / 8);
  if ((e = hipMemcpyAsync(cnt.data(), counts, cnt_bytes, hipMemcpyDeviceToHost, st)) !=
          hipSuccess ||
      (e = hipStreamSynchronize(st)) != hipSuccess)
    return hip_err(ctx, e, "gamma readback");
  uint64_t nr = 0, np = 0;
  for (int k = 0; k < kGammaSlots; ++k) {
    nr += cnt[(size_t)k * 16];
    np += cnt[(size_t)k * 16 + 1];
  }
  if (n_region) *n_region = nr;
  if (n_pass) *n_pass = np;
  return CTD_OK;
}
