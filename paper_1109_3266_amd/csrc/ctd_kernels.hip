// HIP kernels for gfx950 (MI355X): Woodcock photon transport (Jia et al.,
// arXiv 1109.3266, Sec. 2.1-2.2), batch fold and sigma-bar reduction,
// Metropolis-Hastings beamlet chains (Alg. A1), macro-cell set-up and
// microbenchmarks.
//
// Execution model.  One persistent launch per round (per tracking mode: the
// global-majorant and macro-cell steps are separate instantiations).  A round is, for each
// participating case, one batch of histories laid out bin-major over the
// spectrum (Sec. 2.2.5), split into chunks of consecutive history ids.  Each
// 64-lane wave owns one case at a time and a pool of history ids claimed one
// chunk per atomic; lanes are one photon each (Sec. 2.2, one thread per
// photon).  When at least `refill_min` lanes of a wave are idle the wave
// refills them in one step from its source stash in LDS, which the whole wave
// fills by sampling the sources of its pool's next ids at once, so a wave
// keeps ~all lanes busy without sampling on a few lanes at a time, and its
// lanes hold photons of neighbouring ids, i.e. similar energies.  A wave
// that claims a chunk of a different case finishes its live photons first.
//
// Numerics.  Transport is float32.  Every deposit (E - E' of a Compton event,
// E of a photoelectric or cutoff event) and every escape is an exact
// multiple of q = 2^-24 keV for E < 256 keV, so deposits enter the int64 tally
// exactly and incident = deposited + escaped holds exactly in q units.
// Random numbers: Philox4x32-10 keyed by the case seed, counter (k,
// history id lo, hi, 0); k = 0 draws the source.  With the global majorant
// blocks k >= 1 are read two words (a pair) at a time: a Woodcock step takes
// a pair (free path, interaction type), a Compton or Rayleigh scatter the
// pair after its step (polar zeta, azimuth); with MACRO tracking flight k
// takes block k (optical depth, interaction type, zeta, azimuth).  Two more
// streams use
// the fourth counter word: (0, h lo, h hi, 1) the fluence-map beamlet of
// history h (inverse CDF, or trial and acceptance of Alg. A1), and
// (0, c, 0, 2) the starting beamlet of Metropolis-Hastings chain c.
#include <hip/hip_runtime.h>

#include "ctd_bound.h"
#include "ctd_internal.h"

namespace ctd {

// Pointers the step loop dereferences are tagged with the global address
// space so they compile to global_* (not flat_*) memory instructions (the
// tag only exists in the device compilation pass).
#if defined(__HIP_DEVICE_COMPILE__)
#define GLOBAL __attribute__((address_space(1)))
#define LOCAL __attribute__((address_space(3)))
#else
#define GLOBAL
#define LOCAL
#endif

// ---------------------------------------------------------------- helpers

// Tally mode 2: per-wave LDS sub-tally of 2^kCacheBits slots (int32 key +
// uint64 value each, 6 KB per wave), in dynamic shared memory.
constexpr int kCacheBits = 9;
constexpr int kCacheSlots = 1 << kCacheBits;
constexpr int kCacheBytesPerWave = kCacheSlots * (8 + 4);

// Dynamic LDS of a transport workgroup, in this order: a 16-byte header
// (the workgroup's next case); the descriptor of the case the workgroup works
// on and its 256-entry palette or bound-class table (every wave of a
// workgroup works on the same case); deferred kind without the event log, the
// case's coarse bound grid (coarse_cap bytes); per wave, its event counters and
// (other kinds) an 8-byte word per lane (what a lane's waiting scatter needs
// later); in tally mode 2, each wave's sub-tally; per wave, its source
// stash of stash_cap records (stash_cap entry points and energies as float4,
// then stash_cap directions as float4, w = the record's history offset);
// with the coarse grid, per wave, its parked photons (three planes of park_cap
// float4); where the tables fit, the case's majorant nodes (padded to 16 B),
// mu/rho rows (not with the coarse grid: there only collision passes read them)
// and bound-test sums.
constexpr int kWaveAccBytes = (ACC_COUNT * 8 + 15) & ~15;
constexpr int kStashRecBytes = 32;
constexpr int kParkRecBytes = 48;
constexpr int kWaveSlotBytes = kWaveAccBytes + 64 * 8;
constexpr int kWaveCaseBytes = ((int)sizeof(CaseDev) + 15) & ~15;
constexpr int kWgHeaderBytes = 16;
constexpr int kWgCaseOff = kWgHeaderBytes;
constexpr int kWgPalOff = kWgCaseOff + kWaveCaseBytes;
constexpr int kWgSlotsOff = kWgPalOff + 256 * 8;

// a ^ b ^ c in one instruction (gfx950 three-input bitwise op, truth table 0x96)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                          uint32_t k0, uint32_t k1) {
  uint32_t x0 = c0, x1 = c1, x2 = c2, x3 = c3;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)x0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)x2;
    const uint32_t y0 = xor3((uint32_t)(p1 >> 32), x1, k0);
    const uint32_t y2 = xor3((uint32_t)(p0 >> 32), x3, k1);
    x1 = (uint32_t)p1;
    x3 = (uint32_t)p0;
    x0 = y0;
    x2 = y2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return make_uint4(x0, x1, x2, x3);
}

// (2 (r >> 9) + 1) 2^-24 exactly: [1,2) mantissa trick minus (1 - 2^-24).
// The float 1.m with m = r >> 9 is bits [40:9] of the 64-bit {0x7F, r}: one
// v_alignbit_b32 instead of a shift and an or.
__device__ __forceinline__ float unif(uint32_t r) {
  return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, r, 9u)) - 0x1.fffffep-1f;
}

__device__ __forceinline__ float lerpf(float a, float b, float w) { return fmaf(w, b - a, a); }

// sin / cos of a phase given in turns (revolutions), hardware transcendental.
__device__ __forceinline__ float sin_turns(float t) { return __builtin_amdgcn_sinf(t); }
__device__ __forceinline__ float cos_turns(float t) { return __builtin_amdgcn_cosf(t); }

// Inverse-CDF surface mu(zeta, E): one 16-byte cell gives both zeta
// neighbours at both energy neighbours; bilinear, clamped to [-1, 1].
// Q: row 0 of the surfaces; row: energy cell, past the rows of other materials
__device__ __forceinline__ float surface(const GLOBAL float4 *__restrict__ Q, int nz,
                                         uint32_t row, float we, float zeta) {
  const float f = zeta * (float)(nz - 1);
  const int i = min((int)f, nz - 2);
  const float wz = f - (float)i;
  const float4 q = Q[(uint64_t)row * (uint32_t)(nz - 1) + (uint32_t)i];
  const float s0 = lerpf(q.x, q.y, wz);
  const float s1 = lerpf(q.z, q.w, wz);
  return fminf(fmaxf(lerpf(s0, s1, we), -1.0f), 1.0f);
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ void atomic_add_u64(unsigned long long *p, unsigned long long v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The fields the step loop reads, as one wave-uniform record.  It is filled
// with readfirstlane when a wave takes its first chunk of a case, so the
// compiler keeps it in scalar registers; everything else about a case (source
// geometry, the angular surfaces and cutoff used at real scatters, counters,
// log) is read from the workgroup's LDS copy of the full descriptor.
struct StepCase {
  const GLOBAL uint2 *vox;
  const GLOBAL uint8_t *vox8;
  const GLOBAL float4 *mu_rho;
  const GLOBAL float *mu_max;
  // the workgroup's LDS copies of mu_rho and mu_max, or null (read mu_rho,
  // mu_max through the caches)
  const LOCAL float4 *tab;
  const LOCAL float *tabmax;
  const LOCAL float *tabbnd;
  // bound-test sums per material and energy cell (CaseDev::bnd)
  const GLOBAL float *bnd;
  GLOBAL unsigned long long *tally;
  // deposit records (kOutRecords): the workgroup's cursors of the case's
  // voxel buckets and its segment counter in LDS, the record array
  LOCAL unsigned long long *cur;
  LOCAL uint32_t *seg_next;
  GLOBAL uint2 *rec;
  GLOBAL uint32_t *rec_prev;
  uint32_t bbits;
  float fnx, fny, fnz, inv_dx, inv_dy, inv_dz, e0, inv_de;
  int32_t nx, ny, ne, rayleigh, npal;
  // tally mode 2: the wave's LDS sub-tally (slot keys = voxel or -1, values);
  // null in modes 0 and 1
  LOCAL int32_t *ckeys;
  LOCAL unsigned long long *cvals;
  // bound grid of blocks of 2^bshift voxels per edge (ceil(n / 2^bshift)
  // blocks per axis); null: every tentative collision reads its voxel
  const GLOBAL uint8_t *bgrid;
  int32_t bshift;
  // coarse bound grid (in LDS; deferred kind): cell edge
  int32_t cshift;
  uint32_t key0, key1;
};

// Id of the XCD (accelerator complex die) this wave runs on.
__device__ __forceinline__ uint32_t xcc_id() {
  // hwreg(HW_REG_XCC_ID, 0, 16): read-only hardware register
  return __builtin_amdgcn_s_getreg(20 | (0 << 6) | ((16 - 1) << 11)) & 0xFu;
}

template <typename T>
__device__ __forceinline__ GLOBAL T *uniform_ptr(T *p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (GLOBAL T *)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ float uniform_f(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ __forceinline__ int32_t uniform_i(int32_t x) {
  return __builtin_amdgcn_readfirstlane(x);
}

// tally: the batch tally of the round's case; tally_mode 0: as it is; 1, 2:
// this XCD's copy of it; cache: the wave's LDS sub-tally (mode 2) or null;
// bound_shift: the bound grid used (-1: none).
__device__ __forceinline__ StepCase make_step_case(const CaseDev &c, unsigned long long *tally,
                                                   int tally_mode, int bound_shift,
                                                   int coarse_cap, LOCAL unsigned char *cache) {
  StepCase s;
  s.cur = nullptr;
  s.seg_next = nullptr;
  s.rec = nullptr;
  s.rec_prev = nullptr;
  s.bbits = 0;
  s.bgrid = nullptr;
  s.bshift = 0;
  s.cshift = c.coarse && uniform_i(c.ncoarse) <= coarse_cap ? uniform_i(c.cshift) : 31;
  if (bound_shift >= 0 && c.bclass) {
    s.bgrid = uniform_ptr(c.bgrid[bound_shift]);
    s.bshift = uniform_i(c.npal) > 0 ? 0 : bound_shift;
  }
  s.vox = uniform_ptr(c.vox);
  s.vox8 = uniform_ptr(c.vox8);
  s.npal = uniform_i(c.npal);
  s.mu_rho = uniform_ptr(c.mu_rho);
  s.tab = nullptr;
  s.tabmax = nullptr;
  s.tabbnd = nullptr;
  s.bnd = uniform_ptr(c.bnd);
  s.mu_max = uniform_ptr(c.mu_max);
  s.tally = uniform_ptr(tally);
  if (tally_mode) s.tally += (size_t)xcc_id() * (size_t)uniform_i((int32_t)c.V);
  s.cvals = (LOCAL unsigned long long *)cache;
  s.ckeys = cache ? (LOCAL int32_t *)(cache + kCacheSlots * 8) : nullptr;
  s.fnx = uniform_f(c.fnx);
  s.fny = uniform_f(c.fny);
  s.fnz = uniform_f(c.fnz);
  s.inv_dx = uniform_f(c.inv_dx);
  s.inv_dy = uniform_f(c.inv_dy);
  s.inv_dz = uniform_f(c.inv_dz);
  s.e0 = uniform_f(c.e0);
  s.inv_de = uniform_f(c.inv_de);
  s.nx = uniform_i(c.nx);
  s.ny = uniform_i(c.ny);
  s.ne = uniform_i(c.ne);
  s.rayleigh = uniform_i(c.rayleigh);
  s.key0 = (uint32_t)uniform_i((int32_t)c.key0);
  s.key1 = (uint32_t)uniform_i((int32_t)c.key1);
  return s;
}

__device__ __forceinline__ uint64_t lane0_u64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, 0);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), 0);
  return ((uint64_t)hi << 32) | lo;
}

// ------------------------------------------------------------ lane state

// Per-wave event counters in LDS (one slot of ACC_COUNT words per wave),
// bumped with LDS atomics when an event happens and added to the case's
// device counters when the wave switches case or exits.  Keeping them out of
// registers leaves room for more resident waves.  Lanes that add to one word
// take turns in the LDS (half of the CU's cycles on water), so what follows
// from other sums is not counted here: the deposited energy is the sum of the
// batch tallies (k_fold), absorptions and deposits follow from the counts of
// how histories go on and end (water 76.3 -> 71.0 ms per 1e9 histories, the
// pencil beam 15.3 -> 13.1 ms per 2e8).
struct Counters {
  unsigned long long *s;
  __device__ __forceinline__ void add(int i, unsigned long long v) { atomicAdd(s + i, v); }
};

__device__ void flush(Counters &c, unsigned long long *acc, int lane, uint32_t refills) {
  if (lane == 0 && refills) c.add(ACC_N_REFILLS, refills);
  if (lane < ACC_COUNT) {
    const unsigned long long v = atomicExch(c.s + lane, 0ull);
    if (v) atomic_add_u64(acc + lane, v);
  }
}

// Device scope in every tally mode: a per-XCD copy is only updated by waves of
// its XCD, but those belong to many workgroups (on gfx950 both scopes give the
// same atomic instruction, performed at the memory side).
__device__ __forceinline__ void tally_add(const StepCase &S, int32_t vox, unsigned long long q) {
  __hip_atomic_fetch_add(S.tally + vox, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Deposit records (kOutRecords): append (voxel within its bucket, q) to the
// bucket's segment of this workgroup.  A cursor word holds the segment and
// the records appended to it: one LDS add gives a lane its place, unless the
// segment is full.  The lane whose add finds it so first (exactly one per
// segment) takes the workgroup's next segment, links it to the full one and
// installs it, while later lanes add again a bounded number of times.  A lane
// without a slot after that, or in a workgroup without segments left, adds
// straight to the tally.  Against the tally's atomics a deposit costs the wave
// an LDS round trip and an 8-byte store instead of an atomic that the memory
// side performs one by one; no fewer bytes leave the L2, since most lines go
// out before they are full (37 bytes written per record, 32 per atomic; water
// 128x128x100, 1e8 histories: 11.4 ms at 94 % of the memory-side atomic rate,
// 5.2 ms with records, VALU 87 % busy with 60 % of lanes).  The slow
// path's loop condition is the wave's (a ballot), so the installing lane
// always runs inside it.
__device__ __forceinline__ void record_deposit(const StepCase &S, int32_t vox, uint32_t q) {
  LOCAL unsigned long long *cur = S.cur + ((uint32_t)vox >> S.bbits);
  unsigned long long w =
      __hip_atomic_fetch_add(cur, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  if ((uint32_t)w >= kLogSeg) {
    bool todo = true;
    for (int t = 0; __ballot(todo) != 0ull; ++t) {
      if (!todo) continue;
      const bool mine = (uint32_t)w == kLogSeg;
      const uint32_t next = __hip_atomic_fetch_add(S.seg_next, mine ? 1u : 0u, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
      if (next >= S.seg_next[1] || (!mine && t >= 16)) {
        if ((uint32_t)w >= kCursorHigh) {   // (ctd_records.h)
          unsigned long long seen = w + 1ull;
          __hip_atomic_compare_exchange_strong(cur, &seen, cursor_full(w), __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        tally_add(S, vox, q);
        w = kLogSeg;
        todo = false;
      } else if (mine) {
        S.rec_prev[next] = (uint32_t)(w >> 32);
        w = (unsigned long long)next << 32;
        __hip_atomic_store(cur, w | 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        todo = false;
      } else {
        w = __hip_atomic_fetch_add(cur, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        todo = (uint32_t)w >= kLogSeg;
      }
    }
    if ((uint32_t)w == kLogSeg) return;   // it went to the tally
  }
  const uint32_t i = (uint32_t)(w >> 32) * kLogSeg | (uint32_t)w;
  S.rec[i] = make_uint2((uint32_t)vox & ((1u << S.bbits) - 1u), q);
}

// Tally mode 2: add the wave's LDS sub-tally to the case's tally and empty it
// (called by the whole wave, before it changes case and at exit).
__device__ void flush_cache(const StepCase &S, int lane) {
  if (!S.ckeys) return;
  for (int i = lane; i < kCacheSlots; i += 64) {
    const int32_t key = S.ckeys[i];
    if (key >= 0) {
      const unsigned long long v = S.cvals[i];
      if (v) tally_add(S, key, v);
      S.ckeys[i] = -1;
      S.cvals[i] = 0ull;
    }
  }
  // the wave's later deposits (any lane) must see the emptied slots
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ void clear_cache(LOCAL unsigned char *cache, int lane) {
  LOCAL unsigned long long *v = (LOCAL unsigned long long *)cache;
  LOCAL int32_t *k = (LOCAL int32_t *)(cache + kCacheSlots * 8);
  for (int i = lane; i < kCacheSlots; i += 64) {
    v[i] = 0ull;
    k[i] = -1;
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

struct Photon {
  float px, py, pz;   // position, voxel units
  float ux, uy, uz;   // unit direction
  float E;            // keV
  float mumax;        // majorant at E, cm^-1
  float sc;           // ln2 / mumax
  float we;           // energy-grid weight
  int je;             // energy-grid cell
  uint32_t hlo, hhi;  // history id
  uint32_t k;         // random pairs taken (MACRO tracking: flights), flag bits
  uint32_t seq;       // event sequence (debug log only)
  uint32_t ks;        // Woodcock steps taken (debug log only)
  // MACRO tracking: a flight (optical depth tau to spend) may span several
  // calls; its random words for the collision and its current cell persist
  float tau;            // < 0: no flight in progress
  uint32_t ry, rz, rw;
  uint32_t cell;        // x | y << 10 | z << 20; all ones: take it from the position
};

// Photon.k: in the low bits the random pairs the photon has taken (global
// majorant) or its flights (MACRO tracking), kScatBit once the photon has
// scattered, kEndBit once its history has ended (and kGoneBit if it left the
// box) until the wave's next refill step counts it, with the other histories
// that ended meanwhile, kDueBit while a scatter selected
// at a block's second pair waits for the next block (plain steps; the
// voxel, material and process wait in the lane's LDS slot).
constexpr uint32_t kScatBit = 0x80000000u;
constexpr uint32_t kGoneBit = 0x40000000u;
constexpr uint32_t kDueBit = 0x20000000u;
constexpr uint32_t kEndBit = 0x10000000u;
constexpr uint32_t kStepMask = 0x0FFFFFFFu;

// mu/rho rows ti and ti + 1 (energy nodes je, je + 1 of one material): from
// the workgroup's LDS copy (TAB) or through the caches.
template <bool TAB>
__device__ __forceinline__ void table_rows(const StepCase &S, uint32_t ti, float4 &t0, float4 &t1) {
  if constexpr (TAB) {
    t0 = S.tab[ti];
    t1 = S.tab[ti + 1];
  } else {
    t0 = S.mu_rho[ti];
    t1 = S.mu_rho[ti + 1];
  }
}

// Bound-test sum in energy cell j (CaseDev::bnd) of the material whose row is
// the staged class's: an LDS address (TAB) or an index.
template <bool TAB>
__device__ __forceinline__ float bound_sum(const StepCase &S, uint32_t row, int j) {
  if constexpr (TAB) return *(const LOCAL float *)(uintptr_t)(row + 4u * (uint32_t)j);
  else return S.bnd[row + (uint32_t)j];
}

template <bool TAB>
__device__ __forceinline__ void set_energy(Photon &p, const StepCase &S, float E) {
  p.E = E;
  const float f = (E - S.e0) * S.inv_de;
  const int j = min(max((int)f, 0), S.ne - 2);
  p.je = j;
  p.we = f - (float)j;
  if constexpr (TAB)
    p.mumax = lerpf(S.tabmax[j], S.tabmax[j + 1], p.we);
  else
    p.mumax = lerpf(S.mu_max[j], S.mu_max[j + 1], p.we);
  p.sc = 0.69314718055994531f * __builtin_amdgcn_rcpf(p.mumax);
}

// Direction after deflection cos(theta) = mu and azimuth 2 pi t (t in turns).
__device__ __forceinline__ void rotate(Photon &p, float mu, float t) {
  const float st = __builtin_amdgcn_sqrtf(fmaxf(0.0f, (1.0f - mu) * (1.0f + mu)));
  const float sp = sin_turns(t), cp = cos_turns(t);
  const float u = p.ux, v = p.uy, w = p.uz;
  float nu, nv, nw;
  if (fabsf(w) < 1.0f - 1e-5f) {
    const float r = __builtin_amdgcn_sqrtf((1.0f - w) * (1.0f + w));
    const float g = st * __builtin_amdgcn_rcpf(r);
    nu = fmaf(u, mu, g * (u * w * cp - v * sp));
    nv = fmaf(v, mu, g * (v * w * cp + u * sp));
    nw = fmaf(w, mu, -st * cp * r);
  } else {
    nu = st * cp;
    nv = st * sp;
    nw = w >= 0.0f ? mu : -mu;
  }
  const float n = rsqrtf(nu * nu + nv * nv + nw * nw);
  p.ux = nu * n;
  p.uy = nv * n;
  p.uz = nw * n;
}

template <int OUT>
__device__ __forceinline__ void log_event(const CaseDev &G, Photon &p, int type, int64_t vox,
                                          float e, float Eafter) {
  if constexpr (OUT != kOutEvents) return;
  const uint64_t h = ((uint64_t)p.hhi << 32) | p.hlo;
  if (h < G.log_h0 || h >= G.log_h1) return;
  const unsigned long long idx = atomicAdd(G.log_n, 1ull);
  if (idx < G.log_cap) {
    ctd_event ev;
    ev.h = h;
    ev.seq = p.seq;
    ev.k = p.ks;
    ev.type = type;
    ev.reserved = 0;
    ev.vox = vox;
    ev.e = e;
    ev.E = Eafter;
    G.log[idx] = ev;
  }
  p.seq += 1;
}

// Exact tally update: e is a multiple of 2^-24 keV, so q = e * 2^24 is an
// integer (< 2^32 for e < 256 keV) and the int64 sum is exact in any order.
template <int OUT>
__device__ __forceinline__ void deposit(const StepCase &S, const CaseDev &G, Photon &p,
                                        Counters &c, int32_t vox, float e, int type,
                                        float Eafter) {
  const uint32_t q = (uint32_t)(e * kQScale);
  if (q) {
    bool cached = false;
    if constexpr (OUT == kOutRecords) {
      record_deposit(S, vox, q);
      cached = true;
    } else if (S.ckeys) {
      // LDS sub-tally: the slot of vox belongs to the first voxel that took
      // it during this wave's case; other voxels go straight to the tally
      const uint32_t slot = ((uint32_t)vox * 2654435761u) >> (32 - kCacheBits);
      int32_t owner = S.ckeys[slot];
      if (owner == -1) {
        int32_t expected = -1;
        __hip_atomic_compare_exchange_strong(S.ckeys + slot, &expected, vox, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        owner = expected == -1 ? vox : expected;
      }
      if (owner == vox) {
        __hip_atomic_fetch_add(S.cvals + slot, (unsigned long long)q, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WAVEFRONT);
        cached = true;
      }
    }
    if (!cached) tally_add(S, vox, q);
  }
  log_event<OUT>(G, p, type, vox, e, Eafter);
}

// Source photon of history h from spectrum bin j (Sec. 2.2.5-2.2.6): its
// entry point into the voxel box (voxel units) and energy in pe, its unit
// direction in dir.xyz; returns false when the ray misses the box (the photon
// escapes at once).  Its start event is logged here (event 0 of the history).
template <int OUT>
__device__ bool source(const StepCase &S, const CaseDev &G, uint64_t h, int j,
                       const int32_t *__restrict__ mh_beam, uint64_t local, Counters &c,
                       float4 &pe, float4 &dir) {
  Photon p;   // only the history id and log fields are used here
  p.hlo = (uint32_t)h;
  p.hhi = (uint32_t)(h >> 32);
  p.seq = 0;
  p.ks = 0;
  const uint4 r = philox10(0u, p.hlo, p.hhi, 0u, S.key0, S.key1);
  const float E = fmaf(unif(r.x), G.bin_width, ((const GLOBAL float *)G.bin_lo)[j]);
  float sx, sy, sz, dx, dy, dz;
  int beamlet = -1;
  if (G.kind == CTD_GEOM_PENCIL) {
    sx = G.src[0]; sy = G.src[1]; sz = G.src[2];
    dx = G.dir[0]; dy = G.dir[1]; dz = G.dir[2];
  } else {
    float sp, cp, zoff;
    if (G.nproj > 0) {
      // exact in double: 24-bit uniform times an integer < 2^31
      int pi = (int)((double)unif(r.y) * (double)G.nproj);
      pi = min(pi, G.nproj - 1);
      const float4 sc = ((const GLOBAL float4 *)G.proj_sc)[pi];
      sp = sc.x;
      cp = sc.y;
      zoff = sc.z;
    } else {
      const float rel = unif(r.y) * G.arc_turns;     // turns since phi0
      const float t = rel + G.phi0_turns;
      sp = sin_turns(t);
      cp = cos_turns(t);
      zoff = G.z_feed * rel;
    }
    sx = fmaf(G.sad, sp, G.iso[0]);
    sy = fmaf(G.sad, cp, G.iso[1]);
    sz = G.iso[2] + zoff;
    float a, b;
    if (G.fl_n > 0) {
      int I;
      if (G.fl_chains > 0) {
        I = ((const GLOBAL int32_t *)mh_beam)[local];               // Alg. A1 chain step of this history
      } else {
        // beamlet I = min{I : C_I > u F}, decided in FP64 (exact inputs: u has
        // 24 bits, k / 2^gbits <= u exactly, so the guide entry is a lower bound)
        const uint4 r2 = philox10(0u, p.hlo, p.hhi, 1u, S.key0, S.key1);
        const double u = (double)unif(r2.x);
        const double x = u * G.fl_total;
        I = ((const GLOBAL int32_t *)G.fl_guide)[(int)(u * (double)(1 << G.fl_gbits))];
        while (I < G.fl_n - 1 && ((const GLOBAL double *)G.fl_cdf)[I] <= x) ++I;
      }
      const int ib = I / G.fl_na;
      const int ia = I - ib * G.fl_na;
      a = fmaf((float)ia + unif(r.z), G.fl_da, G.a0);
      b = fmaf((float)ib + unif(r.w), G.fl_db, G.b0);
      beamlet = I;
    } else {
      a = fmaf(unif(r.z), G.a1 - G.a0, G.a0);
      b = fmaf(unif(r.w), G.b1 - G.b0, G.b0);
    }
    const float Px = fmaf(a, cp, G.iso[0]);
    const float Py = fmaf(-a, sp, G.iso[1]);
    const float Pz = sz + b;
    const float vx = Px - sx, vy = Py - sy, vz = Pz - sz;
    const float inv = rsqrtf(vx * vx + vy * vy + vz * vz);
    dx = vx * inv; dy = vy * inv; dz = vz * inv;
  }
  c.add(ACC_N_HIST, 1);
  c.add(ACC_Q_INC, (uint32_t)(E * kQScale));
  log_event<OUT>(G, p, 0, beamlet, E, E);
  // slab entry into the box [0, n) in voxel units
  const float Sv[3] = {(sx - G.ox) * S.inv_dx, (sy - G.oy) * S.inv_dy, (sz - G.oz) * S.inv_dz};
  const float D[3] = {dx * S.inv_dx, dy * S.inv_dy, dz * S.inv_dz};
  const float N[3] = {S.fnx, S.fny, S.fnz};
  float tn = -INFINITY, tf = INFINITY;
  bool miss = false;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (D[a] == 0.0f) {
      miss |= (Sv[a] < 0.0f) | (Sv[a] > N[a]);
    } else {
      const float inv = __builtin_amdgcn_rcpf(D[a]);
      const float t1 = (0.0f - Sv[a]) * inv, t2 = (N[a] - Sv[a]) * inv;
      tn = fmaxf(tn, fminf(t1, t2));
      tf = fminf(tf, fmaxf(t1, t2));
    }
  }
  const float tin = fmaxf(tn, 0.0f);
  if (miss || !(tin < tf)) {
    c.add(ACC_N_MISS, 1);
    c.add(ACC_Q_ESC, (uint32_t)(E * kQScale));
    log_event<OUT>(G, p, 6, -1, E, E);
    return false;
  }
  // entry point, kept inside [0, n) against rounding
  // (+ 0.0f turns a -0 into +0 and leaves every other value as it is; a
  // step's fma from a position that is not -0 never gives -0, so positions
  // are never -0: see inside_box)
  pe.x = fminf(fmaxf(fmaf(tin, D[0], Sv[0]), 0.0f), __int_as_float(__float_as_int(N[0]) - 1)) + 0.0f;
  pe.y = fminf(fmaxf(fmaf(tin, D[1], Sv[1]), 0.0f), __int_as_float(__float_as_int(N[1]) - 1)) + 0.0f;
  pe.z = fminf(fmaxf(fmaf(tin, D[2], Sv[2]), 0.0f), __int_as_float(__float_as_int(N[2]) - 1)) + 0.0f;
  pe.w = E;
  dir.x = dx; dir.y = dy; dir.z = dz;
  return true;
}

// Counters of a history that has ended (kEndBit), at the wave's next refill
// step: one pass over all of them instead of one inside each step (water 63.8
// -> 60.4 ms per 1e9 histories, with the voxel layout fixed per instance).
template <int OUT>
__device__ __forceinline__ void count_ended(Photon &p, const CaseDev &G, Counters &c) {
  c.add(ACC_N_STEPS, p.k & kStepMask);
  if (p.k & kGoneBit) {   // left the voxel box with its energy
    c.add(ACC_N_ESCAPES, 1);
    if (!(p.k & kScatBit)) c.add(ACC_N_UNSCATTERED, 1);
    c.add(ACC_Q_ESC, (uint32_t)(p.E * kQScale));
    log_event<OUT>(G, p, 5, -1, p.E, p.E);
  }
  p.k &= ~(kGoneBit | kEndBit);
}

// Outcome of the selection at a tentative collision; kSelPhoto and kSelDone
// end the photon.
constexpr int kSelFict = 0, kSelCompton = 1, kSelRayleigh = 2, kSelPhoto = 3, kSelDone = 4;

// Selection at a tentative collision (Sec. 2.1) in voxel vox of density rho,
// given the mass attenuation coefficients (a, b, cr) = (photoelectric,
// Compton, Rayleigh) interpolated at E and xi = u1 * the majorant:
// photoelectric, Compton, Rayleigh or fictitious by comparing xi with the
// cumulative sums in that order.  A photoelectric absorption deposits E
// locally here.
template <int OUT, bool TAB>
__device__ __forceinline__ int select_process(Photon &p, const StepCase &S, const CaseDev &G,
                                              Counters &c, int32_t vox, float rho, float a,
                                              float b, float cr, float xi) {
  const float mpe = rho * a;
  const float c1 = mpe + rho * b;
  if (xi < mpe) {  // photoelectric: absorb, deposit E locally
    p.k |= kEndBit;
    deposit<OUT>(S, G, p, c, vox, p.E, 1, 0.0f);
    return kSelPhoto;
  }
  if (xi < c1) return kSelCompton;
  if (TAB || S.rayleigh) {
    const float c2 = c1 + rho * cr;
    if (xi < c2) return kSelRayleigh;
  }
  return kSelFict;
}

// Selection in voxel vox of density bits rbits and material m against majorant
// mumax with selection word ry.
template <int OUT, bool TAB>
__device__ __forceinline__ int select_in(Photon &p, const StepCase &S, const CaseDev &G,
                                         Counters &c, int32_t vox, uint32_t rbits, uint32_t m,
                                         uint32_t ry, float mumax) {
  const uint32_t ti = __umul24(m, (uint32_t)S.ne) + (uint32_t)p.je;
  float4 t0, t1;
  table_rows<TAB>(S, ti, t0, t1);
  const float a = lerpf(t0.x, t1.x, p.we), b = lerpf(t0.y, t1.y, p.we);
  // (the staged rows hold 0 for Rayleigh where the case has none)
  const float cr = TAB || S.rayleigh ? lerpf(t0.z, t1.z, p.we) : 0.0f;
  return select_process<OUT, TAB>(p, S, G, c, vox, __uint_as_float(rbits), a, b, cr,
                             unif(ry) * mumax);
}

// Tentative collision at voxel vox against majorant mumax with selection
// word ry: read the voxel (1-byte palette index or 8-byte record) and its
// table rows, then select; m receives the voxel's material.
// LAYOUT: voxels as palette indices or 8-byte records, or as the case has them.
constexpr int kVoxAny = 0, kVoxPalette = 1, kVoxRecord = 2;
template <int OUT, bool TAB, int LAYOUT>
__device__ __forceinline__ int select_at(Photon &p, const StepCase &S, const CaseDev &G,
                                         const LOCAL uint2 *pal, Counters &c, int32_t vox,
                                         uint32_t ry, float mumax, uint32_t &m) {
  uint32_t rbits;
  if (LAYOUT == kVoxPalette || (LAYOUT == kVoxAny && S.npal)) {  // 1-byte index into the workgroup's LDS palette
    const uint32_t i8 = S.vox8[vox];
    rbits = pal[i8].x;
    m = pal[i8].y;
  } else {
    const uint2 rec = S.vox[vox];
    rbits = rec.x;
    m = rec.y;
  }
  return select_in<OUT, TAB>(p, S, G, c, vox, rbits, m, ry, mumax);
}

// Compton (sel = kSelCompton, Sec. 2.2.3) or Rayleigh (Sec. 2.2.2) scatter in
// voxel vox of material m: the polar angle from the process's surface at
// uniform w0, the azimuth from w1; returns false when the photon is done
// (Compton below the cutoff).  Both processes go through the surface lookup
// and the rotation together: most waves have lanes of each, and the rotation
// is half of a scatter (water 60.4 -> 57.2 ms per 1e9 histories, macro-cell
// head 32.8 -> 32.0 ms, six uneven cases 58.8 -> 56.9 ms).
template <int OUT, bool TAB>
__device__ __forceinline__ bool scatter(Photon &p, const StepCase &S, const CaseDev &G,
                                        Counters &c, int sel, int32_t vox, uint32_t m,
                                        uint32_t w0, uint32_t w1) {
  p.k |= kScatBit;
  const bool compton = sel == kSelCompton;
  c.add(compton ? ACC_N_COMPTON : ACC_N_RAYLEIGH, 1);
  // surface fields from the workgroup's LDS copy of the case (read only here)
  const uint32_t mrow = __umul24(m, (uint32_t)(S.ne - 1)) + (uint32_t)p.je;
  const float mu = surface((const GLOBAL float4 *)(compton ? G.comp_quad : G.rayl_quad),
                           compton ? G.nzc : G.nzr,
                           compton && !G.comp_per_mat ? (uint32_t)p.je : mrow, p.we, unif(w0));
  rotate(p, mu, unif(w1));
  if (!compton) {
    log_event<OUT>(G, p, 3, vox, 0.0f, p.E);
    return true;
  }
  const float E = p.E;
  const float Ep = E * __builtin_amdgcn_rcpf(fmaf(E * kInvMeC2, 1.0f - mu, 1.0f));
  deposit<OUT>(S, G, p, c, vox, E - Ep, 2, Ep);  // exact: Ep > E/2 (Sterbenz)
  set_energy<TAB>(p, S, Ep);
  if (Ep < G.e_cut) {
    c.add(ACC_N_CUTOFF, 1);
    p.k |= kEndBit;
    deposit<OUT>(S, G, p, c, vox, Ep, 4, 0.0f);
    return false;
  }
  return true;
}

// 0 <= position < n on each axis, as one unsigned compare of the float bits.
// Positions are never -0 (the entry point is made +0, and a step's fma
// x + s d from an x that is not -0 cannot give -0); for the other floats the
// bits of non-negative values order like the values, while negative values,
// infinities and NaNs (sign bit set, or exponent all ones) compare above
// every finite positive bound -- outside, as the two float compares say.
__device__ __forceinline__ bool inside_box(const Photon &p, const StepCase &S) {
  return (__float_as_uint(p.px) < __float_as_uint(S.fnx)) &
         (__float_as_uint(p.py) < __float_as_uint(S.fny)) &
         (__float_as_uint(p.pz) < __float_as_uint(S.fnz));
}

// Voxel of a position inside the box.
__device__ __forceinline__ int32_t voxel_at(const Photon &p, const StepCase &S) {
  return (int32_t)__umul24(__umul24((uint32_t)p.pz, (uint32_t)S.ny) + (uint32_t)p.py,
                           (uint32_t)S.nx) + (int32_t)(uint32_t)p.px;
}

// Step guard of the global-majorant steps, checked once per block: a photon
// that has taken kStepGuard pairs stops (a runaway history, which
// ctd_read_balance reports as an error); returns false then.
__device__ __forceinline__ bool guard_ok(const Photon &p, Counters &c) {
  const uint32_t P = p.k & kStepMask;
  if (P < kStepGuard) return true;
  c.add(ACC_STEP_GUARD, 1);
  c.add(ACC_N_STEPS, P);
  return false;
}

// Random words of the global-majorant steps: the history's transport blocks
// are read two words (a pair) at a time in order; pair P (the low bits of
// Photon.k count the pairs taken) is words 2 (P mod 2), 2 (P mod 2) + 1 of
// block P / 2 + 1.  A step takes a pair (free path, selection), a Compton or
// Rayleigh scatter the pair after its step (polar angle, azimuth).
template <int OUT>
__device__ __forceinline__ uint4 pair_block(const Photon &p, const StepCase &S, uint32_t P) {
  uint32_t k0 = S.key0, k1 = S.key1;
#if defined(__HIP_DEVICE_COMPILE__)
  // the record-keeping instance recomputes the 18 round keys (scalar adds)
  // instead of holding them over the step loop, where they push its pointers
  // into vector registers (water 57.2 -> 55.9 ms per 1e9; the head, whose step
  // has scalar registers left, 124.6 -> 125.2 ms, keeps them)
  if constexpr (OUT == kOutRecords) asm volatile("" : "+s"(k0), "+s"(k1));
#endif
  return philox10((P >> 1) + 1u, p.hlo, p.hhi, 0u, k0, k1);
}

// One Woodcock step (Sec. 2.1) against the global majorant with words w0
// (free path) and w1 (selection), the tentative collision read from its voxel
// (cases with a bound grid take step_fast and the collision passes instead).
// Returns the selection; a Compton or Rayleigh scatter is left to the
// caller, with the voxel and its material in vox and m.  The caller applies
// the step guard, once per block.
template <int OUT, bool TAB, int LAYOUT>
__device__ __forceinline__ int step(Photon &p, const StepCase &S, const CaseDev &G,
                                    const LOCAL uint2 *pal, Counters &c, uint32_t w0,
                                    uint32_t w1, int32_t &vox, uint32_t &m) {
  p.k += 1;
  if (OUT == kOutEvents) p.ks += 1;
  const float s = -__log2f(unif(w0)) * p.sc;  // -ln(u) / mu_max
  p.px = fmaf(s, p.ux * S.inv_dx, p.px);
  p.py = fmaf(s, p.uy * S.inv_dy, p.py);
  p.pz = fmaf(s, p.uz * S.inv_dz, p.pz);
  const bool inside = inside_box(p, S);
  if (!inside) {
    p.k |= kGoneBit | kEndBit;
    return kSelDone;
  }
  const uint32_t ix = (uint32_t)p.px, iy = (uint32_t)p.py, iz = (uint32_t)p.pz;
  vox = (int32_t)__umul24(__umul24(iz, (uint32_t)S.ny) + iy, (uint32_t)S.nx) + (int32_t)ix;
  return select_at<OUT, TAB, LAYOUT>(p, S, G, pal, c, vox, w1, p.mumax, m);
}

// One Woodcock step with deferred collisions (bound grid present), words w0
// (free path) and w1 (selection): the fast part of step() -- free path,
// move, exit test and the rejection of fictitious collisions by the bound
// grids -- leaving the rest to the wave's next collision pass.  halt stays
// kGoing after a fictitious collision; kWaiting: a tentative collision that
// needs its voxel, w1 kept in u1 for the pass, which selects as step() does;
// kGone: left the box.  The caller applies the step guard, once per block.
// The coarse grid in LDS comes first: a byte per cell, no energy, and most of
// the air and half of the soft tissue's collisions are decided there; only the
// rest read the bound grid, a random byte of 1.3 MB that L1 hardly holds.
constexpr uint32_t kGoing = 0, kWaiting = 1, kGone = 2, kStopped = 3;

template <int OUT, bool TAB>
__device__ __forceinline__ void step_fast(Photon &p, const StepCase &S, const LOCAL uint2 *cls_tab,
                                          const LOCAL uint8_t *coarse,
                                          const GLOBAL uint8_t *bgrid, uint32_t &u1,
                                          uint32_t &halt, uint32_t w0, uint32_t w1) {
  p.k += 1;
  if (OUT == kOutEvents) p.ks += 1;
  const float s = -__log2f(unif(w0)) * p.sc;  // -ln(u) / mu_max
  p.px = fmaf(s, p.ux * S.inv_dx, p.px);
  p.py = fmaf(s, p.uy * S.inv_dy, p.py);
  p.pz = fmaf(s, p.uz * S.inv_dz, p.pz);
  if (!inside_box(p, S)) {
    halt = kGone;
    return;
  }
  const uint32_t ix = (uint32_t)p.px, iy = (uint32_t)p.py, iz = (uint32_t)p.pz;
  if constexpr (OUT == kOutTally) {
    const uint32_t ce = (1u << S.cshift) - 1u;
    const uint32_t cnx = ((uint32_t)S.nx + ce) >> S.cshift, cny = ((uint32_t)S.ny + ce) >> S.cshift;
    const uint32_t cell = __umul24(__umul24(iz >> S.cshift, cny) + (iy >> S.cshift), cnx) +
                          (ix >> S.cshift);
    if ((w1 >> 24) > coarse[cell]) return;
  }
  const uint32_t e = (1u << S.bshift) - 1u;
  const uint32_t bgx = ((uint32_t)S.nx + e) >> S.bshift, bgy = ((uint32_t)S.ny + e) >> S.bshift;
  const uint32_t blk = __umul24(__umul24(iz >> S.bshift, bgy) + (iy >> S.bshift), bgx) +
                       (ix >> S.bshift);
  const uint2 ce = cls_tab[bgrid[blk]];
  if (unif(w1) * p.mumax >= __uint_as_float(ce.x) * bound_sum<TAB>(S, ce.y, p.je)) return;
  u1 = w1;
  halt = kWaiting;
}

// Woodcock tracking with the macro-cell majorant (MACRO tracking).  A flight
// draws its random block (step k) and spends the optical depth tau = -ln(u0)
// cell by cell along the ray; a boundary crossing draws no random number.  A
// call takes at most kMacroCrossings cells and then hands the flight on to
// the next call (tau, the block's remaining words and the cell are kept in
// the photon), so the lanes of a wave advance in similar strides instead of
// all waiting for the longest flight.  Termination: a flight's cell index
// moves one cell per crossing along the direction of travel, so it leaves the
// grid or collides within the cells per axis summed; every call takes at
// least one crossing or ends the flight.
constexpr int kMacroCrossings = 4;

template <int OUT, bool TAB>
__device__ __forceinline__ bool step_macro(Photon &p, const StepCase &S, const CaseDev &G,
                                           const LOCAL uint2 *pal, Counters &c) {
  if (p.tau < 0.0f) {  // a new flight
    p.k += 1;
    if (OUT == kOutEvents) p.ks += 1;
    const uint32_t k0 = p.k & kStepMask;
    if (k0 > kStepGuard) {
      c.add(ACC_STEP_GUARD, 1);
      c.add(ACC_N_STEPS, k0);
      return false;
    }
    const uint4 r = philox10(k0, p.hlo, p.hhi, 0u, S.key0, S.key1);
    p.tau = -__log2f(unif(r.x)) * 0.69314718055994531f;
    p.ry = r.y;
    p.rz = r.z;
    p.rw = r.w;
    p.cell = 0xFFFFFFFFu;
  }
  float tau = p.tau;
  const int ncx = G.mc_nx, ncy = G.mc_ny, ncz = G.mc_nz;
  const float fcs = G.mc_fcs;
  const float Dx = p.ux * S.inv_dx, Dy = p.uy * S.inv_dy, Dz = p.uz * S.inv_dz;
  int cx, cy, cz;
  if (p.cell == 0xFFFFFFFFu) {
    cx = min(max((int)(p.px * G.mc_inv_cs), 0), ncx - 1);
    cy = min(max((int)(p.py * G.mc_inv_cs), 0), ncy - 1);
    cz = min(max((int)(p.pz * G.mc_inv_cs), 0), ncz - 1);
  } else {
    cx = (int)(p.cell & 1023u);
    cy = (int)((p.cell >> 10) & 1023u);
    cz = (int)(p.cell >> 20);
  }
  // the cell majorant factors of the photon's energy band
  const GLOBAL float *fband =
      (const GLOBAL float *)G.mc_f + (size_t)(p.je >> G.mc_shift) * (size_t)G.mc_ncell;
  // per axis, fixed for the call: the face the ray leaves a cell by, the
  // index step, 1/D, and whether the ray moves along the axis at all
  const bool fx = Dx > 0.0f, fy = Dy > 0.0f, fz = Dz > 0.0f;
  const bool mx = Dx != 0.0f, my = Dy != 0.0f, mz = Dz != 0.0f;
  const float rx = __builtin_amdgcn_rcpf(Dx), ry = __builtin_amdgcn_rcpf(Dy),
              rz = __builtin_amdgcn_rcpf(Dz);
  uint32_t crossings = 0;
  float mu_c = 0.0f;
  bool hit = false, out = false;
#pragma unroll
  for (int it = 0; it < kMacroCrossings; ++it) {
    mu_c = fband[(cz * ncy + cy) * ncx + cx] * p.mumax;
    const float x0 = (float)cx * fcs, y0 = (float)cy * fcs, z0 = (float)cz * fcs;
    const float bx = fx ? fminf(x0 + fcs, S.fnx) : x0;
    const float by = fy ? fminf(y0 + fcs, S.fny) : y0;
    const float bz = fz ? fminf(z0 + fcs, S.fnz) : z0;
    const float tx = mx ? fmaxf((bx - p.px) * rx, 0.0f) : INFINITY;
    const float ty = my ? fmaxf((by - p.py) * ry, 0.0f) : INFINITY;
    const float tz = mz ? fmaxf((bz - p.pz) * rz, 0.0f) : INFINITY;
    const float d = fminf(tx, fminf(ty, tz));
    if (tau < mu_c * d) {  // tentative collision inside this cell
      hit = true;
      break;
    }
    tau -= mu_c * d;
    p.px = fmaf(d, Dx, p.px);
    p.py = fmaf(d, Dy, p.py);
    p.pz = fmaf(d, Dz, p.pz);
    ++crossings;
    // the nearest face, ties to x then y (no branches: one index moves)
    const bool ax = tx <= ty && tx <= tz;
    const bool ay = !ax && ty <= tz;
    cx += ax ? (fx ? 1 : -1) : 0;
    cy += ay ? (fy ? 1 : -1) : 0;
    cz += (!ax && !ay) ? (fz ? 1 : -1) : 0;
    out = (unsigned)cx >= (unsigned)ncx || (unsigned)cy >= (unsigned)ncy ||
          (unsigned)cz >= (unsigned)ncz;
    if (out) break;
  }
  if (crossings) c.add(ACC_N_CROSS, crossings);
  if (out) {
    p.tau = -1.0f;
    p.k |= kGoneBit | kEndBit;
    return false;
  }
  if (!hit) {  // the flight goes on in the next call, from this cell
    p.tau = tau;
    p.cell = (uint32_t)cx | ((uint32_t)cy << 10) | ((uint32_t)cz << 20);
    return true;
  }
  p.tau = -1.0f;
  const float s = tau * __builtin_amdgcn_rcpf(mu_c);
  p.px = fmaf(s, Dx, p.px);
  p.py = fmaf(s, Dy, p.py);
  p.pz = fmaf(s, Dz, p.pz);
  // the voxel is taken inside the current cell, whose majorant bounds it
  const int cs = G.mc_cs;
  const int ix = min(max((int)p.px, cx * cs), min(cx * cs + cs, S.nx) - 1);
  const int iy = min(max((int)p.py, cy * cs), min(cy * cs + cs, S.ny) - 1);
  const int iz = min(max((int)p.pz, cz * cs), min(cz * cs + cs, (int)S.fnz) - 1);
  const int32_t vox = (int32_t)__umul24(__umul24((uint32_t)iz, (uint32_t)S.ny) + (uint32_t)iy,
                                         (uint32_t)S.nx) + ix;
  uint32_t m;
  const int sel = select_at<OUT, TAB, kVoxAny>(p, S, G, pal, c, vox, p.ry, mu_c, m);
  if (sel == kSelFict) return true;
  if (sel == kSelPhoto) return false;
  return scatter<OUT, TAB>(p, S, G, c, sel, vox, m, p.rz, p.rw);
}

// Parked photons (deferred kind).  A lane whose collision waits gives its photon
// to the wave's store in LDS and takes another one, so nearly every lane steps
// until pass_min collisions have gathered; then every lane swaps what it holds
// for a waiting photon, the pass runs on a full wave, and the photons swapped
// out are handed to the lanes that next fall idle.  Bound by instruction issue:
// before, 45 of 64 lanes stepped (the others waited or were idle) and a pass
// had 17; now 56 and 63.  With fewer wave-level steps the L2 became the limit
// (28 requests per history, 0.73 per channel and clock, nearly all random bytes
// of the bound grid), which the coarse grid below relieves (6.3 requests).  Head, 1e9 histories: 124.8 ms without both, 122.8 parked
// only, 102.5 with the coarse grid, 88.4 with the states of a lane in one
// register (halt), staged row addresses and passes of 64.
// Three planes of cap 16-byte words per wave; what set_energy derives from the
// energy is derived again.
__device__ __forceinline__ void park(const Photon &p, LOCAL float4 *pl, uint32_t cap, uint32_t i,
                                     uint32_t u1) {
  pl[i] = make_float4(p.px, p.py, p.pz, p.E);
  pl[cap + i] = make_float4(p.ux, p.uy, p.uz, __uint_as_float(u1));
  pl[2 * cap + i] = make_float4(__uint_as_float(p.hlo), __uint_as_float(p.hhi),
                                __uint_as_float(p.k), 0.0f);
}

// ------------------------------------------------------- transport kernel

__device__ __forceinline__ int find_bin(const unsigned long long *__restrict__ prefix, int nbins,
                                        uint64_t local) {
  int lo = 0, hi = nbins - 1;
  while (lo < hi) {  // last bin with prefix[bin] <= local
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= local) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Chunks of round case c, reloaded from the launch table where needed
// rather than kept live across the step loop.
__device__ __forceinline__ uint64_t case_chunk_count(const RoundCase *__restrict__ rcs, int nrc,
                                                     uint64_t total_chunks, int c) {
  return (c + 1 < nrc ? rcs[c + 1].chunk_begin : total_chunks) - rcs[c].chunk_begin;
}

// The home case of workgroup g: the last case whose home workgroups start
// at or before g.
__device__ __forceinline__ int home_case(const RoundCase *__restrict__ rcs, int nrc, uint32_t g) {
  int lo = 0, hi = nrc - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (rcs[mid].wg_lo <= g) lo = mid; else hi = mid - 1;
  }
  return lo;
}

static_assert(sizeof(CaseDev) % 4 == 0 && sizeof(CaseDev) <= 512, "CaseDev copy size");

// Copy a case descriptor and its voxel palette or, for deferred steps, its
// bound-grid class table into the workgroup's LDS (threads copy words; the
// caller's barrier publishes them).  A class holds its density level and the
// row of its material's bound-test sums, at bnd0 + bnd_step * material; the
// mixed class an infinite level, which rejects nothing.
__device__ __forceinline__ void stage_case(CaseDev *dst, uint2 *pal, const CaseDev *src,
                                           uint32_t bnd0, uint32_t bnd_step, bool defer) {
  const uint32_t *s = reinterpret_cast<const uint32_t *>(src);
  uint32_t *d = reinterpret_cast<uint32_t *>(dst);
  for (int i = threadIdx.x; i < (int)(sizeof(CaseDev) / 4); i += blockDim.x) d[i] = s[i];
  const uint2 *sp = src->palette;
  const uint2 *sc = src->bclass;
  if (!defer && __builtin_amdgcn_readfirstlane(src->npal) > 0)
    for (int i = threadIdx.x; i < 256; i += blockDim.x) pal[i] = sp[i];
  else if (defer && sc)
    for (int i = threadIdx.x; i < 256; i += blockDim.x)
      pal[i] = i == (int)kMixedClass ? make_uint2(__float_as_uint(INFINITY), bnd0)
                                     : make_uint2(sc[i].x, bnd0 + __umul24(sc[i].y, bnd_step));
}

// KIND selects the step for every case of the launch (kStepPlain,
// kStepDeferred, kStepMacro, kStepRecord; a round whose cases need different
// steps is split into one launch per step), so each instance carries only its own
// step's registers and a tight loop of its steps between refills.  Every
// instance is held to 96 VGPRs (5 waves per SIMD): the global steps fit
// without spilling, the macro-cell step spills a few words outside its cell
// walk and gains more from the fifth wave hiding its dependent cell/majorant
// loads than the spills cost.
template <int OUT, int KIND, bool TAB>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(5))) k_transport(const RoundCase *__restrict__ rcs, int nrc,
                                                   uint64_t total_chunks,
                                                   unsigned long long *chunk_ctr, int refill_min,
                                                   int chunk, int tally_mode, int bound_shift,
                                                   int defer_min, int tab_n, int tab_ne,
                                                   int stash_cap, int park_cap, int coarse_cap,
                                                   DepositLog dl) {
  extern __shared__ unsigned long long dyn_lds[];   // layout: see kWgSlotsOff
  const int lane = __lane_id();
  const int w = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
  const unsigned long long lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  unsigned char *base = (unsigned char *)dyn_lds;
  int *wg_next = (int *)base;   // the workgroup's next case (header word)
  CaseDev &G = *(CaseDev *)(base + kWgCaseOff);
  uint2 *pal = (uint2 *)(base + kWgPalOff);
  const LOCAL uint2 *pal_lds = (const LOCAL uint2 *)pal;
  constexpr bool kDefer = KIND == kStepDeferred;
  constexpr bool kPark = kDefer && OUT == kOutTally;
  const int slots_off = kWgSlotsOff + (kPark ? coarse_cap : 0);
  constexpr int kSlotBytes = kDefer ? kWaveAccBytes : kWaveSlotBytes;
  LOCAL uint8_t *coarse = (LOCAL uint8_t *)(base + kWgSlotsOff);
  unsigned char *slot = base + slots_off + w * kSlotBytes;
  unsigned char *after_slots = base + slots_off + nw * kSlotBytes;
  LOCAL uint2 *lane_word = (LOCAL uint2 *)(slot + kWaveAccBytes) + lane;
  // staged tables: the majorant nodes and mu/rho rows of the workgroup's
  // current case and its bound-test sums, shared by its waves (room for the
  // round's largest case)
  LOCAL float *tabmax = nullptr;
  LOCAL float4 *tab = nullptr;
  LOCAL float *tabbnd = nullptr;
  unsigned char *after_cache = after_slots + (tally_mode == 2 ? nw * kCacheBytesPerWave : 0);
  LOCAL float4 *st_a = (LOCAL float4 *)(after_cache + w * stash_cap * kStashRecBytes);
  LOCAL float4 *st_b = st_a + stash_cap;
  // deposit records: the header's two words (next segment, end of the
  // workgroup's segments) and the cursors behind the stash
  LOCAL uint32_t *seg_next = (LOCAL uint32_t *)(base + 4);
  unsigned char *after_stash = after_cache + nw * stash_cap * kStashRecBytes;
  LOCAL float4 *pl = (LOCAL float4 *)after_stash + w * 3 * park_cap;
  if constexpr (kPark) after_stash += nw * park_cap * kParkRecBytes;
  LOCAL unsigned long long *cur = (LOCAL unsigned long long *)after_stash;
  if constexpr (OUT == kOutRecords) {
    after_stash += (size_t)dl.cursors * 8;
    if (threadIdx.x == 0) {
      seg_next[0] = 1u + blockIdx.x * dl.seg_per_wg;
      seg_next[1] = seg_next[0] + dl.seg_per_wg;
    }
  }
  if (TAB) {
    tabmax = (LOCAL float *)after_stash;
    tab = (LOCAL float4 *)(tabmax + ((tab_ne + 3) & ~3));
    tabbnd = (LOCAL float *)(tab + (kPark ? 0 : tab_n));
  }

  Counters cnt;
  cnt.s = (unsigned long long *)slot;
  if (lane < ACC_COUNT) cnt.s[lane] = 0ull;
  LOCAL unsigned char *cache =
      tally_mode == 2 ? (LOCAL unsigned char *)after_slots + w * kCacheBytesPerWave : nullptr;
  if (cache) clear_cache(cache, lane);

  // Workgroup g starts on its home case (RoundCase::wg_lo: the case holding
  // chunk g * waves of the round).  The home waves of a case take its first
  // chunks by rank, with no atomic (the launch does not start with every
  // wave queueing on one address); every later claim of case c is
  // home_waves(c) + atomicAdd(counter c).  When a case has no chunk left,
  // the workgroup's waves drain, and the workgroup moves on together to the
  // next case (cyclically) that still has chunks, restaging its tables; it
  // exits when none has.  Results do not depend on this order: each history
  // is a function of its id, and the tallies are exact integer sums.
  int c = home_case(rcs, nrc, blockIdx.x);
  bool home = true;
  StepCase S;
  uint64_t pool_next = 0, pool_end = 0;  // local history indices of case c
  int wbin = 0;                          // bin of pool_next
  // the stash: records [st_pos, st_n) are sources not yet handed out, of the
  // histories st_base + their offsets
  uint64_t st_base = 0;
  uint32_t st_pos = 0, st_n = 0;
  bool first = true, claims_done = false;
  uint32_t refills = 0;
  Photon p;
  p.k = 0;
  bool alive = false;
  // deferred collisions: whether the lane's photon waits for a pass, and its
  // selection word; the wave's parked photons, n_wait that wait in [0, n_wait)
  // and n_on that go on in [park_cap - n_on, park_cap)
  bool wait = false;
  uint32_t u1 = 0, n_wait = 0, n_on = 0;
  const uint32_t pass_min = kPark && park_cap > 0
                                ? min((uint32_t)park_cap - 4u, 4u * (uint32_t)defer_min)
                                : (uint32_t)max(defer_min, 1);
  for (;;) {
    if (TAB) {
      const CaseDev *cd = rcs[c].cd;
      const int n_rows = cd->nmat * cd->ne, n_e = cd->ne;
      const float4 *src = cd->mu_rho;
      const float *srcm = cd->mu_max;
      const bool rayl = cd->rayleigh != 0;
      if constexpr (!kPark) {
        for (int i = threadIdx.x; i < n_rows; i += blockDim.x) {
          float4 r = src[i];
          if (!rayl) r.z = 0.0f;
          tab[i] = r;
        }
      }
      for (int i = threadIdx.x; i < n_e; i += blockDim.x) tabmax[i] = srcm[i];
      const float *srcb = cd->bnd;
      const int n_b = cd->nmat * (n_e - 1);
      for (int i = threadIdx.x; i < n_b; i += blockDim.x) tabbnd[i] = srcb[i];
    }
    const uint32_t cells = (uint32_t)rcs[c].cd->ne - 1u;
    if (TAB) stage_case(&G, pal, rcs[c].cd, (uint32_t)(uintptr_t)tabbnd, 4u * cells, kDefer);
    else stage_case(&G, pal, rcs[c].cd, 0u, cells, kDefer);
    if constexpr (kPark) {
      // (without a grid, or room for it: one cell that rejects nothing)
      const CaseDev *cd = rcs[c].cd;
      const uint32_t *src = cd->ncoarse <= coarse_cap ? (const uint32_t *)cd->coarse : nullptr;
      const int nw4 = src ? (cd->ncoarse + 3) / 4 : 1;
      for (int i = threadIdx.x; i < nw4; i += blockDim.x)
        ((LOCAL uint32_t *)coarse)[i] = src ? src[i] : 255u;
    }
    if constexpr (OUT == kOutRecords) {
      const int nb = (int)rcs[c].buckets;
      for (int i = threadIdx.x; i < nb; i += blockDim.x) cur[i] = (unsigned long long)kLogSeg;
    }
    __syncthreads();   // case and tables staged before any wave steps
    pool_next = pool_end = 0;
    wbin = 0;
    st_pos = st_n = 0;
    first = true;
    claims_done = false;
    refills = 0;

    for (;;) {
      const unsigned long long dead = __ballot(!alive);
      const int ndead = __popcll(dead);
      // deferred kind: a pass comes first where enough collisions wait (it
      // takes the idle lanes), otherwise every idle lane gets a photon
      bool due = false, hand_out = ndead == 64 || ndead >= refill_min;
      if constexpr (kDefer) {
        due = n_wait + (uint32_t)__popcll(__ballot(alive && wait)) >= pass_min;
        if (!alive && (p.k & kEndBit)) count_ended<OUT>(p, G, cnt);
        hand_out = dead != 0ull && !due;
      }
      if (hand_out) {
        // counters of the histories that ended since the last refill step
        if constexpr (!kDefer)
          if (!alive && (p.k & kEndBit)) count_ended<OUT>(p, G, cnt);
        // idle lanes take the stash's records in order, lowest lanes first;
        // an empty stash is refilled from the pool (a chunk of case c is
        // claimed when the pool is empty) with the sources of the pool's
        // next stash_cap ids, sampled by the whole wave at once
        const bool want = !alive;
        const uint32_t rank = (uint32_t)__popcll(dead & lt_mask);
        uint32_t filled = 0;
        if constexpr (kPark) {
          if (n_on) {
            filled = min((uint32_t)ndead, n_on);
            if (want && rank < filled) {
              const uint32_t i = (uint32_t)park_cap - n_on + rank;
              const float4 a = pl[i], b = pl[park_cap + i], d = pl[2 * park_cap + i];
              p.px = a.x; p.py = a.y; p.pz = a.z;
              p.ux = b.x; p.uy = b.y; p.uz = b.z;
              p.hlo = __float_as_uint(d.x);
              p.hhi = __float_as_uint(d.y);
              p.k = __float_as_uint(d.z);
              set_energy<TAB>(p, S, a.w);
              alive = true;
            }
            n_on -= filled;
          }
        }
        for (;;) {
          if constexpr (kPark)
            if (filled == (uint32_t)ndead) break;
          if (st_pos < st_n) {
            const uint32_t take = min((uint32_t)ndead - filled, st_n - st_pos);
            if (want && rank >= filled && rank < filled + take) {
              const uint32_t i = st_pos + (rank - filled);
              const float4 a = st_a[i], b = st_b[i];
              const uint64_t h = rcs[c].h_begin + st_base + __float_as_uint(b.w);
              p.hlo = (uint32_t)h;
              p.hhi = (uint32_t)(h >> 32);
              p.k = 0;
              p.seq = OUT == kOutEvents ? 1u : 0u;   // event 0 (the start) was logged at sampling
              p.ks = 0;
              p.tau = -1.0f;
              p.px = a.x; p.py = a.y; p.pz = a.z;
              p.ux = b.x; p.uy = b.y; p.uz = b.z;
              set_energy<TAB>(p, S, a.w);
              alive = true;
            }
            st_pos += take;
            filled += take;
            if (filled == (uint32_t)ndead) break;
          }
          while (pool_next >= pool_end && !claims_done) {
            uint64_t t;
            if (home && first) {
              t = (uint64_t)__builtin_amdgcn_readfirstlane(
                  (blockIdx.x - rcs[c].wg_lo) * (uint32_t)nw + (uint32_t)w);
            } else {
              unsigned long long a = 0;
              if (lane == 0) a = atomicAdd(chunk_ctr + c, 1ull);
              t = rcs[c].home_waves + lane0_u64(a);
            }
            if (t >= case_chunk_count(rcs, nrc, total_chunks, c)) {
              claims_done = true;
              break;
            }
            const uint64_t lo = t * (uint64_t)chunk;
            const uint64_t hi = min(lo + (uint64_t)chunk, rcs[c].n);
            // the wave's step constants at its first chunk; a wave's claims
            // of one case increase, so later bin searches start from the last
            if (first) {
              S = make_step_case(G, rcs[c].tally, tally_mode, bound_shift, coarse_cap, cache);
              if constexpr (OUT == kOutRecords) {
                S.cur = cur;
                S.seg_next = seg_next;
                S.rec = (GLOBAL uint2 *)dl.rec;
                S.rec_prev = (GLOBAL uint32_t *)dl.prev;
                S.bbits = uniform_i((int32_t)rcs[c].bucket_bits);
              }
              S.tab = tab;
              S.tabmax = tabmax;
              S.tabbnd = tabbnd;
              wbin = find_bin(rcs[c].prefix, G.nbins, lo);
            }
            first = false;
            pool_next = lo;
            pool_end = hi;
          }
          if (pool_next >= pool_end) break;   // nothing left to hand out
          // sample: lane l takes pool id pool_next + l; the records of the
          // photons that enter the box are stored compacted, in id order
          const RoundCase &R = rcs[c];
          const uint32_t ng = (uint32_t)min((uint64_t)stash_cap, pool_end - pool_next);
          const uint64_t local = pool_next + (uint64_t)lane;
          bool ok = false;
          float4 pe, dir;
          if ((uint32_t)lane < ng) {
            int j = wbin;
            const GLOBAL unsigned long long *pre = (const GLOBAL unsigned long long *)R.prefix;
            while (j + 1 < G.nbins && local >= pre[j + 1]) ++j;
            ok = source<OUT>(S, G, R.h_begin + local, j, R.beamlets, local, cnt, pe, dir);
          }
          const unsigned long long okm = __ballot(ok);
          __builtin_amdgcn_wave_barrier();   // the last records were read
          if (ok) {
            const uint32_t i = (uint32_t)__popcll(okm & lt_mask);
            dir.w = __uint_as_float((uint32_t)lane);
            st_a[i] = pe;
            st_b[i] = dir;
          }
          __builtin_amdgcn_wave_barrier();   // records written before any lane reads them
          st_base = pool_next;
          st_pos = 0;
          st_n = (uint32_t)__popcll(okm);
          pool_next += ng;
          if (pool_next < pool_end) {
            const GLOBAL unsigned long long *pre = (const GLOBAL unsigned long long *)R.prefix;
            while (wbin + 1 < G.nbins && pool_next >= pre[wbin + 1]) ++wbin;
          }
        }
        if (filled > 0) refills += 1;
      }
      if (__ballot(alive) == 0ull && (!kPark || n_wait == 0)) {
        // case c done for this wave
        if (claims_done && pool_next >= pool_end && st_pos >= st_n) break;
        continue;
      }
      if constexpr (KIND == kStepMacro) {
        // one call per pass of the loop: a tight loop of macro-cell calls
        // spills more than it saves
        if (alive) alive = step_macro<OUT, TAB>(p, S, G, pal_lds, cnt);
      } else if constexpr (KIND == kStepDeferred) {
        const unsigned long long on = __ballot(alive && !wait);
        if (due || on == 0ull) {
          // collision pass: the waiting collisions of the wave, once pass_min
          // have gathered or nothing else is left to do
          // the waiting photons' voxel records, asked for as early as possible
          uint2 rec = make_uint2(0u, 0u);
          if (alive && wait) rec = S.vox[voxel_at(p, S)];
          if constexpr (kPark) {
            if (n_wait) {
              // lanes without a waiting collision take the parked ones, idle
              // lanes first; the others park the photon they held
              const unsigned long long idle = __ballot(!alive);
              const uint32_t n_idle = (uint32_t)__popcll(idle);
              const uint32_t n_take = min(n_wait, n_idle + (uint32_t)__popcll(on));
              const uint32_t r = alive ? n_idle + (uint32_t)__popcll(on & lt_mask)
                                       : (uint32_t)__popcll(idle & lt_mask);
              const bool take = !(alive && wait) && r < n_take;
              const bool keep = take && alive;
              const uint32_t in = n_wait - 1u - r;
              const uint32_t out = (uint32_t)park_cap - n_on - 1u - (r - n_idle);
              float4 a;
              __builtin_amdgcn_wave_barrier();
              if (take) a = pl[in];
              __builtin_amdgcn_wave_barrier();
              if (keep) pl[out] = make_float4(p.px, p.py, p.pz, p.E);
              if (take) {
                p.px = a.x; p.py = a.y; p.pz = a.z;
                rec = S.vox[voxel_at(p, S)];
                set_energy<TAB>(p, S, a.w);
                a = pl[park_cap + in];
              }
              __builtin_amdgcn_wave_barrier();
              if (keep) pl[park_cap + out] = make_float4(p.ux, p.uy, p.uz, 0.0f);
              if (take) {
                p.ux = a.x; p.uy = a.y; p.uz = a.z;
                u1 = __float_as_uint(a.w);
                a = pl[2 * park_cap + in];
              }
              __builtin_amdgcn_wave_barrier();
              if (keep)
                pl[2 * park_cap + out] = make_float4(__uint_as_float(p.hlo), __uint_as_float(p.hhi),
                                                     __uint_as_float(p.k), 0.0f);
              if (take) {
                p.hlo = __float_as_uint(a.x);
                p.hhi = __float_as_uint(a.y);
                p.k = __float_as_uint(a.z);
                alive = true;
                wait = true;
              }
              __builtin_amdgcn_wave_barrier();
              n_wait -= n_take;
              n_on += n_take > n_idle ? n_take - n_idle : 0u;
            }
          }
          if (alive && wait) {
            const uint32_t P = p.k & kStepMask;
            uint32_t m;
            const int32_t vox = voxel_at(p, S);
            const int sel = select_in<OUT, TAB && !kPark>(p, S, G, cnt, vox, rec.x, rec.y, u1,
                                                          p.mumax);
            m = rec.y;
            if (sel == kSelPhoto) {
              alive = false;
            } else if (sel != kSelFict) {   // the scatter takes the next pair
              const uint4 q = pair_block<OUT>(p, S, P);
              const bool odd = (P & 1u) != 0u;
              p.k += 1;
              alive = scatter<OUT, TAB>(p, S, G, cnt, sel, vox, m, odd ? q.z : q.x,
                                              odd ? q.w : q.y);
            }
          }
          wait = false;
          continue;
        }
        // fast steps until refill_min more lanes have stopped (or every lane): a
        // tight loop in which a photon's direction, energy and tables stay put;
        // one block serves two steps (a photon at an odd pair takes one)
        const int quit = max(__popcll(on) - refill_min, 0);
        // the bound grid's address in scalar registers
        const GLOBAL uint8_t *bg = uniform_ptr(S.bgrid);
        uint32_t halt = alive && !wait ? kGoing : ~0u;
        for (;;) {
          if (halt == kGoing) {
            if (!guard_ok(p, cnt)) {
              halt = kStopped;
            } else {
              const uint32_t P = p.k & kStepMask;
              const uint4 r = pair_block<OUT>(p, S, P);
              if ((P & 1u) == 0u)
                step_fast<OUT, TAB>(p, S, pal_lds, coarse, bg, u1, halt, r.x, r.y);
              if (halt == kGoing)
                step_fast<OUT, TAB>(p, S, pal_lds, coarse, bg, u1, halt, r.z, r.w);
            }
          }
          if (__popcll(__ballot(halt == kGoing)) <= quit) break;
        }
        if (halt == kWaiting) wait = true;
        if (halt == kGone || halt == kStopped) alive = false;
        if (halt == kGone) p.k |= kGoneBit | kEndBit;
        if constexpr (kPark) {   // park what waits, as far as there is room
          const unsigned long long pm = __ballot(alive && wait);
          const uint32_t room = (uint32_t)park_cap - n_wait - n_on;
          const uint32_t r = (uint32_t)__popcll(pm & lt_mask);
          __builtin_amdgcn_wave_barrier();
          if (alive && wait && r < room) {
            park(p, pl, (uint32_t)park_cap, n_wait + r, u1);
            alive = false;
            wait = false;
          }
          __builtin_amdgcn_wave_barrier();
          n_wait += min((uint32_t)__popcll(pm), room);
        }
      } else {
        // steps until a refill is due, one block per pass of the loop: its
        // first pair takes a step (and its second pair that step's scatter)
        // or the scatter a photon left waiting; its second pair takes the
        // next step, whose scatter then waits for the next block.  A photon
        // starts every pass at an even pair.
        constexpr int kLayout = KIND == kStepPlain ? kVoxPalette : kVoxRecord;
        for (;;) {
          if (alive && (alive = guard_ok(p, cnt))) {
            const uint4 r = pair_block<OUT>(p, S, p.k & kStepMask);
            int sel;
            int32_t vox = 0;
            uint32_t m = 0, w0 = r.z, w1 = r.w;
            if (p.k & kDueBit) {   // the waiting scatter takes the first pair
              const uint2 lw = *lane_word;
              vox = (int32_t)lw.x;
              m = lw.y & 0xFFFFu;
              sel = (int)(lw.y >> 16);
              p.k &= ~kDueBit;
              w0 = r.x;
              w1 = r.y;
            } else {
              sel = step<OUT, TAB, kLayout>(p, S, G, pal_lds, cnt, r.x, r.y, vox, m);
            }
            if (sel == kSelCompton || sel == kSelRayleigh) {
              p.k += 1;
              alive = scatter<OUT, TAB>(p, S, G, cnt, sel, vox, m, w0, w1);
            } else if (sel >= kSelPhoto) {
              alive = false;
            }
            if (alive && (p.k & 1u)) {   // the block's second pair: a step
              sel = step<OUT, TAB, kLayout>(p, S, G, pal_lds, cnt, r.z, r.w, vox, m);
              if (sel == kSelCompton || sel == kSelRayleigh) {
                *lane_word = make_uint2((uint32_t)vox, m | ((uint32_t)sel << 16));
                p.k |= kDueBit;
              } else if (sel >= kSelPhoto) {
                alive = false;
              }
            }
          }
          if (64 - __popcll(__ballot(alive)) >= refill_min) break;
        }
      }
    }
    if (!first) {   // the wave ran histories of case c
      flush(cnt, G.acc, lane, refills);
      flush_cache(S, lane);
    }
    // every wave of the workgroup has drained case c: pick the next case
    // with chunks left, scanning cyclically from c + 1 (c itself last)
    __syncthreads();
    if constexpr (OUT == kOutRecords) {
      // the case's cursors are final: the heads of this workgroup's chains
      const int nb = (int)rcs[c].buckets;
      unsigned long long *head = dl.head + (size_t)blockIdx.x * dl.buckets + rcs[c].bucket0;
      for (int i = threadIdx.x; i < nb; i += blockDim.x) head[i] = cur[i];
    }
    if (threadIdx.x == 0) {
      int nxt = -1;
      for (int i = 1; i <= nrc && nxt < 0; ++i) {
        const int d = c + i < nrc ? c + i : c + i - nrc;
        const uint64_t taken =
            rcs[d].home_waves +
            __hip_atomic_load(chunk_ctr + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (taken < case_chunk_count(rcs, nrc, total_chunks, d)) nxt = d;
      }
      *wg_next = nxt;
    }
    __syncthreads();
    c = __builtin_amdgcn_readfirstlane(*wg_next);   // uniform: scalar from here on
    home = false;
    if (c < 0) break;
  }
}

// Sum a round's deposit records into the batch tallies.  Workgroup (bucket,
// slice) keeps the bucket's voxels as 64-bit sums in LDS, walks the record
// chains that the slice's transport workgroups left for the bucket (16 lanes
// per chain, a segment at a time, so short chains of a small round still fill
// the waves' loads), then adds its non-zero sums to the tally.  Bound by
// reading the records: 2.04 GB (1e8 water histories) in 0.41 ms, 4.9 TB/s.
__global__ void __launch_bounds__(1024) k_collect(const RoundCase *__restrict__ rcs, int nrc,
                                                  DepositLog dl, int wgs, int slices) {
  extern __shared__ unsigned long long tile[];
  const uint32_t gb = blockIdx.x / (uint32_t)slices;
  const int slice = (int)(blockIdx.x - gb * (uint32_t)slices);
  int lo = 0, hi = nrc - 1;
  while (lo < hi) {   // last case whose first bucket is at or before gb
    const int mid = (lo + hi + 1) >> 1;
    if (rcs[mid].bucket0 <= gb) lo = mid; else hi = mid - 1;
  }
  const RoundCase &rc = rcs[lo];
  const int64_t v0 = (int64_t)(gb - rc.bucket0) << rc.bucket_bits;
  const int nv = (int)min((int64_t)1 << rc.bucket_bits, rc.cd->V - v0);
  for (int i = threadIdx.x; i < nv; i += blockDim.x) tile[i] = 0ull;
  __syncthreads();
  const uint32_t sub = threadIdx.x & 15u;
  const int w1 = (int)((int64_t)wgs * (slice + 1) / slices);
  for (int w = (int)((int64_t)wgs * slice / slices) + (int)(threadIdx.x >> 4); w < w1;
       w += blockDim.x >> 4) {
    const unsigned long long h = dl.head[(size_t)w * dl.buckets + gb];
    uint32_t seg = (uint32_t)(h >> 32), n = min((uint32_t)h, kLogSeg);
    while (seg) {
      const uint32_t nxt = dl.prev[seg];
      const uint4 *r = (const uint4 *)(dl.rec + (size_t)seg * kLogSeg) + sub;
      uint4 d[kLogSeg / 32];
#pragma unroll
      for (uint32_t k = 0; k < kLogSeg / 32; ++k)
        if (32u * k + 2u * sub < n) d[k] = r[16 * k];
#pragma unroll
      for (uint32_t k = 0; k < kLogSeg / 32; ++k) {
        const uint32_t i = 32u * k + 2u * sub;
        if (i < n) atomicAdd(&tile[d[k].x], (unsigned long long)d[k].y);
        if (i + 1u < n) atomicAdd(&tile[d[k].z], (unsigned long long)d[k].w);
      }
      n = kLogSeg;
      seg = nxt;
    }
  }
  __syncthreads();
  unsigned long long *t = rc.tally + v0;
  for (int i = threadIdx.x; i < nv; i += blockDim.x) {
    const unsigned long long v = tile[i];
    if (v == 0ull) continue;
    if (slices == 1) t[i] += v;
    else atomic_add_u64(t + i, v);
  }
}

// MACRO tracking set-up: per cell of cs^3 voxels and material, the largest
// density (float bits; densities are >= 0 so their bits order like values).
__global__ void __launch_bounds__(256) k_cell_max(const uint2 *__restrict__ vox, int nx, int ny,
                                                  int64_t V, int cs, int ncx, int ncy, int M,
                                                  unsigned int *__restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += stride) {
    const uint2 rec = vox[v];
    if (rec.x == 0u || (int)rec.y >= M) continue;
    const int x = (int)(v % nx);
    const int64_t t = v / nx;
    const int y = (int)(t % ny), z = (int)(t / ny);
    const int64_t cell = ((int64_t)(z / cs) * ncy + y / cs) * ncx + x / cs;
    atomicMax(out + cell * M + rec.y, rec.x);
  }
}

// The same with one block per cell, for cells of kCellBlock voxels per edge and
// more: the maxima meet in LDS and every entry of out is written (256x256x160,
// 16-voxel cells: 853 us with an atomic per voxel on few addresses, 22 us now).
constexpr int kCellBlock = 8;
__global__ void __launch_bounds__(256) k_cell_max_block(const uint2 *__restrict__ vox, int nx,
                                                        int ny, int nz, int cs, int ncx, int ncy,
                                                        int M, unsigned int *__restrict__ out) {
  __shared__ unsigned int top[256];
  if ((int)threadIdx.x < M) top[threadIdx.x] = 0u;
  __syncthreads();
  const int cx = (int)(blockIdx.x % (unsigned)ncx);
  const int row = (int)(blockIdx.x / (unsigned)ncx);
  const int x0 = cx * cs, y0 = (row % ncy) * cs, z0 = (row / ncy) * cs;
  const int wx = min(cs, nx - x0), wy = min(cs, ny - y0), wz = min(cs, nz - z0);
  unsigned int cur = 0u, hi = 0u;   // the thread's current material
  for (int i = threadIdx.x; i < wx * wy * wz; i += blockDim.x) {
    const int x = i % wx, t = i / wx;
    const uint2 r = vox[((int64_t)(z0 + t / wy) * ny + (y0 + t % wy)) * nx + (x0 + x)];
    if (r.y != cur) {
      if (hi && (int)cur < M) atomicMax(&top[cur], hi);
      cur = r.y;
      hi = 0u;
    }
    hi = max(hi, r.x);
  }
  if (hi && (int)cur < M) atomicMax(&top[cur], hi);
  __syncthreads();
  if ((int)threadIdx.x < M) out[(int64_t)blockIdx.x * M + threadIdx.x] = top[threadIdx.x];
}

// Coarse bound grid: one block per cell of 2^shift voxels per edge, the byte of
// the cell's largest share rho f[m] (ctd_bound.h).  Reads every voxel once, rows
// of the cell coalesced.
__global__ void __launch_bounds__(256) k_coarse(const uint2 *__restrict__ vox, int nx, int ny,
                                                int nz, int shift, int ncx, int ncy,
                                                const float *__restrict__ f,
                                                uint8_t *__restrict__ out) {
  __shared__ float top[4];
  const int cx = (int)(blockIdx.x % (unsigned)ncx);
  const int row = (int)(blockIdx.x / (unsigned)ncx);
  const int cs = 1 << shift;
  const int x0 = cx * cs, y0 = (row % ncy) * cs, z0 = (row / ncy) * cs;
  const int wx = min(cs, nx - x0), wy = min(cs, ny - y0), wz = min(cs, nz - z0);
  float share = 0.0f;
  for (int i = threadIdx.x; i < wx * wy * wz; i += blockDim.x) {
    const int x = i % wx, t = i / wx;
    const uint2 r = vox[((int64_t)(z0 + t / wy) * ny + (y0 + t % wy)) * nx + (x0 + x)];
    if (r.x) share = fmaxf(share, __uint_as_float(r.x) * f[r.y]);
  }
  for (int d = 32; d > 0; d >>= 1) share = fmaxf(share, __shfl_xor(share, d));
  if ((threadIdx.x & 63) == 0) top[threadIdx.x >> 6] = share;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < 4; ++i) share = fmaxf(share, top[i]);
    out[blockIdx.x] = coarse_byte(share);
  }
}

// Bound grid: one lane per block of 2^shift voxels per edge.  A block whose
// voxels share one material m gets the first of m's density levels (ascending
// in cls[range[m].x ...]) that is at or above the block's largest density;
// the last level is m's largest density over the phantom, so one exists.
// Densities are >= 0 and sign-clear, so their bits order like their values.
// Bound by reading the records (256x256x160, 1-voxel blocks: 172 us with a
// linear search of the levels in global memory, 53 us now).
__global__ void __launch_bounds__(256) k_block_class(const uint2 *__restrict__ vox, int nx, int ny,
                                                     int nz, int shift, int bx, int by,
                                                     int64_t nblocks,
                                                     const uint2 *__restrict__ cls,
                                                     const int2 *__restrict__ range,
                                                     uint8_t *__restrict__ out) {
  __shared__ uint32_t level[256];
  __shared__ int2 rng[256];
  for (int i = threadIdx.x; i < 256; i += blockDim.x) {
    level[i] = cls[i].x;
    rng[i] = range[i];
  }
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int B = 1 << shift;
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < nblocks; b += stride) {
    const int x0 = (int)(b % bx) * B;
    const int64_t t = b / bx;
    const int y0 = (int)(t % by) * B, z0 = (int)(t / by) * B;
    const int x1 = min(x0 + B, nx), y1 = min(y0 + B, ny), z1 = min(z0 + B, nz);
    uint32_t m = vox[((int64_t)z0 * ny + y0) * nx + x0].y, rmax = 0u;
    bool mixed = false;
    for (int z = z0; z < z1; ++z)
      for (int y = y0; y < y1; ++y)
        for (int x = x0; x < x1; ++x) {
          const uint2 r = vox[((int64_t)z * ny + y) * nx + x];
          mixed |= r.y != m;
          rmax = max(rmax, r.x);
        }
    uint32_t c = kMixedClass;
    if (!mixed) {
      int lo = rng[m].x, hi = lo + rng[m].y - 1;   // the last level is high enough
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (level[mid] >= rmax) hi = mid; else lo = mid + 1;
      }
      c = (uint32_t)lo;
    }
    out[b] = (uint8_t)c;
  }
}

// Alg. A1 (Metropolis-Hastings) on logical chains: lane c advances chain c
// over its histories h = c (mod C) of [h_begin, h_begin + n) in increasing h.
// Step of history h: trial J = floor(u0 N_f) and zeta = u1 from the second
// source block; move to J when zeta f_I < f_J (exact in FP64: 24-bit
// operands).  A chain's first history (h = c) starts from a beamlet drawn
// from the counter (0, c_lo, c_hi, 2).
__global__ void __launch_bounds__(256) k_mh_fill(const float *__restrict__ f, int n_f, int C,
                                                 uint64_t h_begin, uint64_t n, uint32_t key0,
                                                 uint32_t key1, int32_t *__restrict__ state,
                                                 int32_t *__restrict__ out) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= C) return;
  const uint64_t Cu = (uint64_t)C;
  const uint64_t r = h_begin % Cu;
  uint64_t h = h_begin + (((uint64_t)c + Cu - r) % Cu);
  const uint64_t end = h_begin + n;
  if (h >= end) return;
  int I;
  if (h < Cu) {
    const uint4 r0 = philox10(0u, (uint32_t)c, 0u, 2u, key0, key1);
    I = min((int)((double)unif(r0.x) * (double)n_f), n_f - 1);
  } else {
    I = state[c];
  }
  double fI = (double)f[I];
  for (; h < end; h += Cu) {
    const uint4 r2 = philox10(0u, (uint32_t)h, (uint32_t)(h >> 32), 1u, key0, key1);
    const int J = min((int)((double)unif(r2.x) * (double)n_f), n_f - 1);
    const double fJ = (double)f[J];
    if ((double)unif(r2.y) * fI < fJ) {
      I = J;
      fI = fJ;
    }
    out[h - h_begin] = I;
  }
  state[c] = I;
}

// --------------------------------------------------------------- fold etc.

// S1 += T_b, S2 += T_b^2 (128-bit), T_b = 0 (Sec. 2.2.1 batch statistics) for
// each batch b of a launch in order: batch 0 in T, the exact sum of its
// ncopies per-XCD copies, the others in `more` ([nbatch - 1][V], one copy).
// The sums are read and written once for all of them; each block adds what it
// folded to its words of the deposited energy (kAccDeposited).  Block 0 also folds the
// counters into their 128-bit totals; every block records the largest S1 and
// S2 high word it produced (overflow headroom; both only grow with b).
__global__ void __launch_bounds__(256) k_fold(unsigned long long *__restrict__ T, int ncopies,
                                              unsigned long long *__restrict__ more, int nbatch,
                                              long long *__restrict__ S1,
                                              unsigned long long *__restrict__ S2, int64_t V,
                                              unsigned long long *__restrict__ acc) {
  __shared__ unsigned long long m1[256], m2[256], ms[256];
  if (blockIdx.x == 0 && threadIdx.x < ACC_COUNT) {
    const unsigned long long v = acc[threadIdx.x];
    if (v) {
      unsigned long long *tot = acc + kAccTotal + 2 * threadIdx.x;
      const unsigned long long lo = tot[0] + v;
      tot[1] += (lo < v) ? 1ull : 0ull;
      tot[0] = lo;
      acc[threadIdx.x] = 0ull;
    }
  }
  unsigned long long mx1 = 0ull, mx2 = 0ull, dep = 0ull;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < V; i += stride) {
    unsigned long long t = 0ull;
    for (int c = 0; c < ncopies; ++c) {
      const unsigned long long v = T[(int64_t)c * V + i];
      if (v) {
        t += v;
        T[(int64_t)c * V + i] = 0ull;
      }
    }
    unsigned long long sum = t, lo = t * t, hi = __umul64hi(t, t);
    for (int b = 1; b < nbatch; ++b) {
      const unsigned long long v = more[(int64_t)(b - 1) * V + i];
      if (v == 0ull) continue;
      more[(int64_t)(b - 1) * V + i] = 0ull;
      sum += v;
      const unsigned long long plo = v * v;
      lo += plo;
      hi += __umul64hi(v, v) + (lo < plo ? 1ull : 0ull);
    }
    if (sum == 0ull) continue;
    dep += sum;
    const long long s1 = S1[i] + (long long)sum;
    S1[i] = s1;
    const unsigned long long nlo = S2[2 * i] + lo;
    const unsigned long long nhi = S2[2 * i + 1] + hi + (nlo < lo ? 1ull : 0ull);
    S2[2 * i] = nlo;
    S2[2 * i + 1] = nhi;
    mx1 = max(mx1, (unsigned long long)s1);
    mx2 = max(mx2, nhi);
  }
  m1[threadIdx.x] = mx1;
  m2[threadIdx.x] = mx2;
  ms[threadIdx.x] = dep;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      m1[threadIdx.x] = max(m1[threadIdx.x], m1[threadIdx.x + o]);
      m2[threadIdx.x] = max(m2[threadIdx.x], m2[threadIdx.x + o]);
      ms[threadIdx.x] += ms[threadIdx.x + o];
    }
    __syncthreads();
  }
  // Atomics on one address serialize at the memory side, so a block whose
  // maximum does not exceed the recorded one skips its atomic.  The recorded
  // maxima only grow (until the host clears them between launches), so a
  // stale read can only add an atomic, never drop a needed one.
  if (threadIdx.x == 0) {
    // the block's part of the deposited energy, 128 bits (its own words; the
    // batches of a launch together stay below 2^63)
    unsigned long long *q = acc + kAccDeposited + 2 * blockIdx.x;
    const unsigned long long lo = q[0] + ms[0];
    q[1] += lo < ms[0] ? 1ull : 0ull;
    q[0] = lo;
    const unsigned long long r1 =
        __hip_atomic_load(acc + kAccMaxS1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long r2 =
        __hip_atomic_load(acc + kAccMaxS2Hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (m1[0] > r1) atomicMax(acc + kAccMaxS1, m1[0]);
    if (m2[0] > r2) atomicMax(acc + kAccMaxS2Hi, m2[0]);
  }
}

// Largest XCC id over all workgroups (read-only hardware register).
__global__ void k_xcc_probe(unsigned int *out) {
  if (threadIdx.x == 0) atomicMax(out, xcc_id());
}

// Pack (mat, rho) into 8-byte voxel records; per-material max and min
// density (as float bits, which order like the values for rho >= 0; the min
// stored complemented so that all-zero memory is its neutral start), voxel
// counts, max material id, a count of bad densities, and the distinct records
// while there are at most 256 (kPack*: k_pack_clear's layout).
//
// A thread keeps the statistics of its current material in registers and adds
// them to the block's when the material changes; a block keeps its distinct
// records in an LDS hash table, looked up when a thread's record changes, and
// adds them to the device's table at its end.  The table is given up (kPackOver)
// at the 257th record, or where a probe finds no room: after that nothing more
// is looked up.  Bound by the 13 bytes per voxel.
constexpr int kLocalSlots = 512;
constexpr unsigned long long kNoRecord = ~0ull;   // material ids are below 256

__device__ __forceinline__ uint32_t record_hash(unsigned long long k) {
  return ((uint32_t)k ^ (uint32_t)(k >> 32) * 0x9E3779B9u) * 2654435761u >> 16;
}

// Whether `key` is in the table afterwards; *count grows by the keys added.
__device__ bool record_insert(unsigned long long *tab, uint32_t slots, unsigned int *count,
                              unsigned long long key) {
  uint32_t h = record_hash(key) & (slots - 1u);
  for (uint32_t t = 0; t < slots; ++t, h = (h + 1u) & (slots - 1u)) {
    unsigned long long k = __hip_atomic_load(tab + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (k == kNoRecord) {
      k = atomicCAS(tab + h, kNoRecord, key);
      if (k == kNoRecord) {
        atomicAdd(count, 1u);
        return true;
      }
    }
    if (k == key) return true;
  }
  return false;
}

// Clears the statistics and looks at kPackSample voxels spread over the grid:
// where those already hold more than 256 records (a phantom with density
// noise), k_pack's blocks need not each fill their table to find out
// (256x256x160 with noise: k_pack 200 us without, 69 us with it).
constexpr int kPackSample = 2048;
__global__ void __launch_bounds__(256) k_pack_clear(const uint8_t *__restrict__ mat,
                                                    const float *__restrict__ rho, int64_t V,
                                                    unsigned int *stats) {
  __shared__ unsigned long long lkey[kLocalSlots];
  __shared__ unsigned int lcount, lover;
  for (int i = threadIdx.x; i < kPackKeys; i += blockDim.x) stats[i] = 0u;
  unsigned long long *keys = (unsigned long long *)(stats + kPackKeys);
  for (int i = threadIdx.x; i < kPackSlots; i += blockDim.x) keys[i] = kNoRecord;
  for (int i = threadIdx.x; i < kLocalSlots; i += blockDim.x) lkey[i] = kNoRecord;
  if (threadIdx.x == 0) lcount = lover = 0u;
  __syncthreads();
  for (int i = threadIdx.x; i < kPackSample; i += blockDim.x) {
    const int64_t v = (int64_t)((double)V * ((double)i / kPackSample));
    const float r = rho[v] == 0.0f ? 0.0f : rho[v];
    const unsigned long long key = (unsigned long long)mat[v] << 32 | __float_as_uint(r);
    if (__hip_atomic_load(&lcount, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > 256u) break;
    if (!record_insert(lkey, kLocalSlots, &lcount, key)) lover = 1u;
  }
  __syncthreads();
  if (threadIdx.x == 0 && (lover || lcount > 256u)) stats[kPackOver] = 1u;
}

__global__ void __launch_bounds__(256) k_pack(const uint8_t *__restrict__ mat,
                                              const float *__restrict__ rho,
                                              uint2 *__restrict__ vox, int64_t V,
                                              unsigned int *stats) {
  __shared__ unsigned int lmax[256], lcnt[256], lmin[256];
  __shared__ unsigned long long lkey[kLocalSlots];
  __shared__ unsigned int lmat, lbad, lcount, lover;
  for (int i = threadIdx.x; i < 256; i += blockDim.x) { lmax[i] = 0u; lcnt[i] = 0u; lmin[i] = 0u; }
  for (int i = threadIdx.x; i < kLocalSlots; i += blockDim.x) lkey[i] = kNoRecord;
  if (threadIdx.x == 0) {
    lmat = lbad = lcount = 0u;
    lover = __hip_atomic_load(stats + kPackOver, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  unsigned int mymat = 0u, mybad = 0u;
  unsigned int cur = 0u, n = 0u, hi = 0u, lo = 0u;   // the current material's statistics
  unsigned long long last = kNoRecord;
  auto settle = [&]() {
    if (!n) return;
    atomicAdd(&lcnt[cur], n);
    if (hi) atomicMax(&lmax[cur], hi);
    if (lo) atomicMax(&lmin[cur], lo);
  };
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < V; i += stride) {
    const unsigned int m = mat[i];
    // -0.0 is stored as +0.0: the per-material extremes below (and the cell
    // maxima of MACRO tracking and the bound classes) order densities by
    // their float bits, which only match their values for sign-clear floats
    const float r = rho[i] == 0.0f ? 0.0f : rho[i];
    const bool ok = (r >= 0.0f) && (r <= 3.4e38f);
    const uint32_t bits = __float_as_uint(r);
    vox[i] = make_uint2(bits, m);
    if (m != cur) {
      settle();
      cur = m;
      n = hi = lo = 0u;
    }
    mymat = max(mymat, m);
    n += 1u;
    if (ok) {
      hi = max(hi, bits);
      lo = max(lo, ~bits);
    } else {
      mybad += 1u;
    }
    const unsigned long long key = (unsigned long long)m << 32 | bits;
    if (key != last) {
      last = key;
      // (at most 256 keys and one more per thread: the probe always ends)
      if (!__hip_atomic_load(&lover, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
        if (!record_insert(lkey, kLocalSlots, &lcount, key) ||
            __hip_atomic_load(&lcount, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > 256u)
          __hip_atomic_store(&lover, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  }
  settle();
  atomicMax(&lmat, mymat);
  if (mybad) atomicAdd(&lbad, mybad);
  __syncthreads();
  for (int i = threadIdx.x; i < 256; i += blockDim.x) {
    if (lmax[i]) atomicMax(&stats[i], lmax[i]);
    if (lcnt[i]) atomicAdd(&stats[256 + i], lcnt[i]);
    if (lmin[i]) atomicMax(&stats[kPackMin + i], lmin[i]);
  }
  if (threadIdx.x == 0) {
    atomicMax(&stats[kPackMat], lmat);
    if (lbad) atomicAdd(&stats[kPackBad], lbad);
  }
  if (lover) {
    if (threadIdx.x == 0) atomicMax(&stats[kPackOver], 1u);
    return;
  }
  unsigned long long *keys = (unsigned long long *)(stats + kPackKeys);
  for (int i = threadIdx.x; i < kLocalSlots; i += blockDim.x) {
    const unsigned long long key = lkey[i];
    if (key == kNoRecord) continue;
    if (!record_insert(keys, kPackSlots, &stats[kPackCount], key)) atomicMax(&stats[kPackOver], 1u);
  }
}

// Palette index of every voxel: the position of its record among the n
// ascending keys.
__global__ void __launch_bounds__(256) k_palette_index(const uint2 *__restrict__ vox, int64_t V,
                                                       const unsigned long long *__restrict__ keys,
                                                       int n, uint8_t *__restrict__ out) {
  __shared__ unsigned long long key[256];
  for (int i = threadIdx.x; i < n; i += blockDim.x) key[i] = keys[i];
  __syncthreads();
  unsigned long long last = kNoRecord;
  int at = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < V; i += stride) {
    const uint2 r = vox[i];
    const unsigned long long k = (unsigned long long)r.y << 32 | r.x;
    if (k != last) {
      last = k;
      int lo = 0, hi = n - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key[mid] >= k) hi = mid; else lo = mid + 1;
      }
      at = lo;
    }
    out[i] = (uint8_t)at;
  }
}

__global__ void __launch_bounds__(256) k_zero(unsigned long long *p, size_t n) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0ull;
}

// sigma-bar, deterministic two-level reductions (fixed grid and block; the
// partials of a level are taken up by all threads of a block, 1e3 dependent
// loads of one thread held k_sigma_sum at 73 us and k_sigma_final at 92 us on
// 1.6e6 voxels, now 13 and 5 us).
__device__ __forceinline__ bool voxel_dose(const long long *s1, const uint2 *vox, int64_t i,
                                           double rho_min, double &d, double &rho) {
  rho = (double)__uint_as_float(vox[i].x);
  if (!(rho >= rho_min) || rho <= 0.0) return false;
  d = (double)s1[i] / rho;
  return true;
}

__global__ void __launch_bounds__(256) k_sigma_max(const long long *s1, const uint2 *vox,
                                                   int64_t V, double rho_min, double *part) {
  __shared__ double sm[256];
  double m = 0.0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < V; i += stride) {
    double d, r;
    if (voxel_dose(s1, vox, i, rho_min, d, r)) m = fmax(m, d);
  }
  sm[threadIdx.x] = m;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sm[0];
}

__global__ void __launch_bounds__(256) k_sigma_sum(const long long *s1,
                                                   const unsigned long long *s2,
                                                   const uint2 *vox, int64_t V, uint32_t nb,
                                                   double rho_min, double frac, int kind,
                                                   const double *part_max, int nparts,
                                                   double *part) {
  __shared__ double ss[256], sc[256];
  double top = 0.0;
  for (int b = threadIdx.x; b < nparts; b += blockDim.x) top = fmax(top, part_max[b]);
  ss[threadIdx.x] = top;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) ss[threadIdx.x] = fmax(ss[threadIdx.x], ss[threadIdx.x + o]);
    __syncthreads();
  }
  const double dmax = ss[0];
  __syncthreads();   // ss is taken again below
  const double nbd = (double)nb;
  double sum = 0.0, count = 0.0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < V; i += stride) {
    double d, rho;
    if (!voxel_dose(s1, vox, i, rho_min, d, rho)) continue;
    if (!(d > frac * dmax) || dmax <= 0.0) continue;
    const double S1 = (double)s1[i];
    const double S2 = (double)s2[2 * i + 1] * 18446744073709551616.0 + (double)s2[2 * i];
    const double var_t = fmax(nbd * S2 - S1 * S1, 0.0) / (nbd * nbd * (nbd - 1.0));
    const double s = sqrt(var_t) * nbd / rho;  // same scale as d = S1 / rho
    sum += (kind == CTD_SIGMA_PAPER) ? s / dmax : s / d;
    count += 1.0;
  }
  ss[threadIdx.x] = sum;
  sc[threadIdx.x] = count;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      ss[threadIdx.x] += ss[threadIdx.x + o];
      sc[threadIdx.x] += sc[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = ss[0];
    part[2 * blockIdx.x + 1] = sc[0];
  }
}

__global__ void __launch_bounds__(256) k_sigma_final(const double *part, int nparts,
                                                     const double *part_max, double *out) {
  __shared__ double ss[256], sc[256], sm[256];
  double s = 0.0, c = 0.0, m = 0.0;
  for (int b = threadIdx.x; b < nparts; b += blockDim.x) {
    s += part[2 * b];
    c += part[2 * b + 1];
    m = fmax(m, part_max[b]);
  }
  ss[threadIdx.x] = s;
  sc[threadIdx.x] = c;
  sm[threadIdx.x] = m;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      ss[threadIdx.x] += ss[threadIdx.x + o];
      sc[threadIdx.x] += sc[threadIdx.x + o];
      sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + o]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = sc[0] > 0.0 ? ss[0] / sc[0] : INFINITY;
    out[1] = sc[0];
    out[2] = sm[0];
  }
}

// ---------------------------------------------------------------- readout

// (nb S2 - S1^2) exactly in 192-bit unsigned arithmetic, returned as double.
__device__ double var_numerator(unsigned long long s1, unsigned long long hi,
                                unsigned long long lo, uint32_t nb) {
  const unsigned long long n = nb;
  const unsigned long long a0 = lo * n, m0 = hi * n;
  const unsigned long long a1 = m0 + __umul64hi(lo, n);
  const unsigned long long a2 = __umul64hi(hi, n) + (a1 < m0 ? 1ull : 0ull);
  const unsigned long long b0 = s1 * s1, b1 = __umul64hi(s1, s1);
  const unsigned long long r0 = a0 - b0, br0 = a0 < b0 ? 1ull : 0ull;
  const unsigned long long r1 = a1 - b1 - br0;
  const unsigned long long br1 = (a1 < b1 || (a1 - b1) < br0) ? 1ull : 0ull;
  if (a2 < br1) return 0.0;  // cannot happen for consistent sums
  const unsigned long long r2 = a2 - br1;
  return (double)r2 * 0x1p128 + (double)r1 * 0x1p64 + (double)r0;
}

// Dose and variance of the mean of voxels [v0, v0 + n) into out[0, n) and
// out[n, 2n) (pinned host memory).  vol_kg: voxel volume times 1e-3; n_hist
// and per_batch: histories of all batches and of one.  Bound by the link the
// 16 bytes per voxel leave by (256x256x160: 168 MB, 3 ms at 57 GB/s; the call
// takes 4.6 ms with the copies into fresh pages overlapped, against 159 ms for
// copying the sums and computing on one host thread).
__global__ void __launch_bounds__(256) k_read_dose(const long long *__restrict__ s1,
                                                   const unsigned long long *__restrict__ s2,
                                                   const uint2 *__restrict__ vox, int64_t v0,
                                                   int n, double vol, double n_hist,
                                                   double per_batch, uint32_t nb,
                                                   double *__restrict__ out) {
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const int64_t v = v0 + i;
    const double mass_kg = (double)__uint_as_float(vox[v].x) * vol * 1e-3;
    double dose = 0.0, var = 0.0;
    if (mass_kg > 0.0) {
      const double conv = 1.602176634e-16 / (16777216.0 * mass_kg);  // q -> Gy
      dose = (double)s1[v] / n_hist * conv;
      const double num =
          var_numerator((unsigned long long)s1[v], s2[2 * v + 1], s2[2 * v], nb);
      const double var_t = num / ((double)nb * nb * (double)(nb - 1));
      var = var_t / (per_batch * per_batch) * conv * conv;
    }
    out[i] = dose;
    out[n + i] = var;
  }
}

// The exact sums of voxels [v0, v0 + n) as three planes out[0, n) = S1,
// out[n, 2n) = high and out[2n, 3n) = low words of S2 (pinned host memory).
__global__ void __launch_bounds__(256) k_read_tally(const unsigned long long *__restrict__ s1,
                                                    const unsigned long long *__restrict__ s2,
                                                    int64_t v0, int n,
                                                    unsigned long long *__restrict__ out) {
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const int64_t v = v0 + i;
    out[i] = s1[v];
    out[n + i] = s2[2 * v + 1];
    out[2 * (int64_t)n + i] = s2[2 * v];
  }
}

// ------------------------------------------------------- microbenchmarks
// Peaks the transport is measured against: streaming copy, random 64-bit
// atomics (no return), atomics into 64 hot words, random 8-byte gathers.
// Addresses come from a 32-bit integer hash of the operation index.

__device__ __forceinline__ uint32_t mix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352dU;
  x ^= x >> 15;
  x *= 0x846ca68bU;
  x ^= x >> 16;
  return x;
}

__global__ void __launch_bounds__(256) k_mb_copy(const uint4 *__restrict__ a,
                                                 uint4 *__restrict__ b, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    b[i] = a[i];
}

__global__ void __launch_bounds__(256) k_mb_atomic(unsigned long long *__restrict__ t,
                                                   uint32_t mask_or_n, int hot, int64_t ops) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ops; i += stride) {
    const uint32_t h = mix32((uint32_t)i);
    const uint32_t idx = hot ? (h & 63u) : (uint32_t)(((uint64_t)h * mask_or_n) >> 32);
    __hip_atomic_fetch_add(t + idx, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__global__ void __launch_bounds__(256) k_mb_gather(const uint2 *__restrict__ v, uint32_t n,
                                                   int64_t ops, uint32_t *out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  uint32_t acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ops; i += stride) {
    const uint32_t idx = (uint32_t)(((uint64_t)mix32((uint32_t)i ^ acc) * n) >> 32);
    const uint2 r = v[idx];
    acc += r.x ^ r.y;
  }
  if (acc == 0x12345678u) out[0] = acc;  // keeps the loads live
}

// ------------------------------------------------ static round table

// The launch table of ctd_run_batches_static.  Host code never passes this
// name to a kernel (on the host it is only a stand-in for the symbol): the
// device address comes from static_scratch_address(), once per device.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// One block writes the round's RoundCase, the bin prefix sums and a zero
// chunk counter into the table (all later work on the stream reads them).
__global__ void __launch_bounds__(256) k_static_round_setup(unsigned char *table,
                                                            StaticRoundArgs a) {
  unsigned long long *pre = (unsigned long long *)(table + kStaticPrefixOff);
  for (int i = threadIdx.x; i <= a.nbins; i += blockDim.x) pre[i] = a.prefix[i];
  unsigned long long *ctr = (unsigned long long *)(table + kStaticCounterOff);
  if (threadIdx.x < 32) ctr[threadIdx.x] = 0ull;
  if (threadIdx.x == 0) {
    RoundCase *rc = (RoundCase *)table;
    rc->cd = a.cd;
    rc->prefix = pre;
    rc->h_begin = a.h_begin;
    rc->n = a.n;
    rc->chunk_begin = 0;
    rc->beamlets = a.beamlets;
    rc->tally = a.tally;
    rc->bucket0 = rc->buckets = rc->bucket_bits = 0;
    rc->wg_lo = 0;
    rc->home_waves = a.home_waves;
  }
}

// ---------------------------------------------------------------- launchers

static int check_launch() { return hipGetLastError() == hipSuccess ? 0 : -1; }

int static_scratch_address(void **out) {
  *out = nullptr;
  return hipGetSymbolAddress(out, HIP_SYMBOL(scratch)) == hipSuccess && *out ? 0 : -1;
}

int launch_static_round_setup(void *table, const StaticRoundArgs &args, void *stream) {
  if (args.nbins < 1 || args.nbins > kStaticMaxBins) return -1;
  hipLaunchKernelGGL(k_static_round_setup, dim3(1), dim3(256), 0, (hipStream_t)stream,
                     (unsigned char *)table, args);
  return check_launch();
}

int launch_transport(const RoundCase *rc_dev, int nrc, uint64_t total_chunks,
                     unsigned long long *chunk_ctr, const LaunchCfg &cfg, int out,
                     const DepositLog &dl, int step_kind, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  // stage the tables (room for the round's largest case) only where the
  // workgroup's LDS then still allows the resident workgroups the grid is
  // sized for, with the largest source stash (64, 32 or 16 records per wave)
  // that fits beside them; without the tables, the largest stash that fits
  // (16 at least).  Deferred launches take with them the coarse bound grid and
  // the largest store of parked photons that fits (72: a pass finds a photon
  // for each of 64 lanes; head 1e9 histories 90.9 ms with 64, 88.4 with 72),
  // or the coarse grid alone, or neither.
  const int cursors = out == kOutRecords ? dl.cursors : 0;
  const bool parks = step_kind == kStepDeferred && out == kOutTally;
  int tab_n = cfg.tab_n, cap = 0, park_cap = 0, coarse_cap = parks ? kCoarseCells : 0;
  const auto bytes = [&](int n, int stash) {
    return transport_lds_bytes(cfg.block, cfg.tally_mode, n, cfg.tab_ne, stash, cursors,
                               parks ? park_cap : -1, coarse_cap);
  };
  if (parks && tab_n > 0 && cfg.defer_min > 0) {
    for (int pc : {72, 64, 48, 32}) {
      park_cap = pc;
      if (bytes(tab_n, 64) <= cfg.lds_budget) cap = 64;
      else if (bytes(tab_n, 32) <= cfg.lds_budget) cap = 32;
      if (cap) break;
    }
    if (!cap) park_cap = 0;
  }
  if (tab_n > 0) {
    for (int c = 64; c >= 16 && !cap; c >>= 1)
      if (bytes(tab_n, c) <= cfg.lds_budget) cap = c;
    if (!cap) tab_n = 0;
  }
  if (!cap) {
    cap = 16;
    if (bytes(0, cap) > cfg.lds_budget) coarse_cap = parks ? 16 : 0;
    for (int c = 64; c > 16 && cap == 16; c >>= 1)
      if (bytes(0, c) <= cfg.lds_budget) cap = c;
  }
  const size_t lds = bytes(tab_n, cap);
  using Kern = void (*)(const RoundCase *, int, uint64_t, unsigned long long *, int, int, int,
                        int, int, int, int, int, int, int, DepositLog);
#define CTD_KIND(OUT, KIND) {k_transport<OUT, KIND, false>, k_transport<OUT, KIND, true>}
  static const Kern kerns[3][kStepKinds][2] = {
      {CTD_KIND(kOutTally, kStepPlain), CTD_KIND(kOutTally, kStepDeferred),
       CTD_KIND(kOutTally, kStepMacro), CTD_KIND(kOutTally, kStepRecord)},
      {CTD_KIND(kOutEvents, kStepPlain), CTD_KIND(kOutEvents, kStepDeferred),
       CTD_KIND(kOutEvents, kStepMacro), CTD_KIND(kOutEvents, kStepRecord)},
      {CTD_KIND(kOutRecords, kStepPlain), {nullptr, nullptr}, {nullptr, nullptr},
       {nullptr, nullptr}}};
#undef CTD_KIND
  if (step_kind < 0 || step_kind >= kStepKinds || out < kOutTally || out > kOutRecords)
    return -1;
  const Kern kern = kerns[out][step_kind][tab_n > 0 ? 1 : 0];
  if (!kern) return -1;
  hipLaunchKernelGGL(kern, dim3(cfg.grid), dim3(cfg.block), lds, s, rc_dev, nrc, total_chunks,
                     chunk_ctr, cfg.refill_min, cfg.chunk, cfg.tally_mode, cfg.bound_shift,
                     cfg.defer_min, tab_n, tab_n > 0 ? cfg.tab_ne : 0, cap, park_cap,
                     coarse_cap, dl);
  return check_launch();
}

int launch_collect(const RoundCase *rc_dev, int nrc, const DepositLog &dl, int wgs,
                   int tile_voxels, int slices, void *stream) {
  hipLaunchKernelGGL(k_collect, dim3((unsigned)dl.buckets * (unsigned)slices), dim3(1024),
                     (size_t)tile_voxels * 8, (hipStream_t)stream, rc_dev, nrc, dl, wgs, slices);
  return check_launch();
}

size_t transport_lds_bytes(int block, int tally_mode, int tab_n, int tab_ne, int stash_cap,
                           int cursors, int park_cap, int coarse_cap) {
  const size_t nw = (size_t)(block / 64);
  size_t b = kWgSlotsOff + nw * kWaveSlotBytes + (tally_mode == 2 ? nw * kCacheBytesPerWave : 0);
  b += nw * (size_t)stash_cap * kStashRecBytes + (size_t)cursors * 8;
  // majorant nodes, mu/rho rows and (room for) the bound-test sums
  if (tab_n > 0) b += (size_t)((tab_ne + 3) & ~3) * 4 + (size_t)tab_n * (park_cap < 0 ? 20 : 4);
  if (park_cap >= 0) b += coarse_cap - nw * (kWaveSlotBytes - kWaveAccBytes);
  if (park_cap > 0) b += nw * (size_t)park_cap * kParkRecBytes;
  return b;
}

bool transport_lds_fits(int block, int tally_mode, int device) {
  int lim = 0;
  if (hipDeviceGetAttribute(&lim, hipDeviceAttributeMaxSharedMemoryPerBlock, device) !=
      hipSuccess) {
    (void)hipGetLastError();  // not a launch error: leave nothing for check_launch
    return false;
  }
  return transport_lds_bytes(block, tally_mode, 0, 0, 16, 0, -1, 0) <= (size_t)lim;
}

static int grid_for(int64_t n, int block, int cap) {
  int64_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (int)g;
}

int launch_fold(unsigned long long *tally, int ncopies, unsigned long long *more, int nbatch,
                long long *s1, unsigned long long *s2, int64_t V, unsigned long long *acc,
                void *stream) {
  // 1024 groups stream the arrays at full rate and keep the per-group
  // maximum records (two loads, at most two atomics each) few
  hipLaunchKernelGGL(k_fold, dim3(grid_for(V, 256, kFoldBlocks)), dim3(256), 0, (hipStream_t)stream,
                     tally, ncopies, more, nbatch, s1, s2, V, acc);
  return check_launch();
}

int launch_xcc_probe(unsigned int *out, int blocks, void *stream) {
  hipLaunchKernelGGL(k_xcc_probe, dim3(blocks), dim3(64), 0, (hipStream_t)stream, out);
  return check_launch();
}

int launch_pack(const uint8_t *mat, const float *rho, uint2 *vox, int64_t V,
                unsigned int *stats, void *stream) {
  hipLaunchKernelGGL(k_pack_clear, dim3(1), dim3(256), 0, (hipStream_t)stream, mat, rho, V, stats);
  hipLaunchKernelGGL(k_pack, dim3(grid_for(V, 256, 2048)), dim3(256), 0, (hipStream_t)stream,
                     mat, rho, vox, V, stats);
  return check_launch();
}

int launch_palette_index(const uint2 *vox, int64_t V, const unsigned long long *keys, int n,
                         uint8_t *out, void *stream) {
  if (V <= 0 || n < 1 || n > 256) return -1;
  hipLaunchKernelGGL(k_palette_index, dim3(grid_for(V, 256, 2048)), dim3(256), 0,
                     (hipStream_t)stream, vox, V, keys, n, out);
  return check_launch();
}

int launch_cell_max(const uint2 *vox, int nx, int ny, int nz, int cs, int ncx, int ncy, int M,
                    unsigned int *out, void *stream) {
  const int64_t V = (int64_t)nx * ny * nz;
  if (V <= 0) return 0;
  const int64_t cells = (int64_t)ncx * ncy * ((nz + cs - 1) / cs);
  if (cs >= kCellBlock && M <= 256 && cells <= 0x7fffffff) {
    hipLaunchKernelGGL(k_cell_max_block, dim3((unsigned)cells), dim3(256), 0, (hipStream_t)stream,
                       vox, nx, ny, nz, cs, ncx, ncy, M, out);
    return check_launch();
  }
  hipLaunchKernelGGL(k_cell_max, dim3(grid_for(V, 256, 8192)), dim3(256), 0, (hipStream_t)stream,
                     vox, nx, ny, V, cs, ncx, ncy, M, out);
  return check_launch();
}

int launch_coarse(const uint2 *vox, int nx, int ny, int nz, int shift, const float *f,
                  uint8_t *out, void *stream) {
  const int e = (1 << shift) - 1;
  const int cx = (nx + e) >> shift, cy = (ny + e) >> shift, cz = (nz + e) >> shift;
  if ((int64_t)cx * cy * cz > kCoarseCells || nx < 1 || ny < 1 || nz < 1) return -1;
  hipLaunchKernelGGL(k_coarse, dim3((unsigned)(cx * cy * cz)), dim3(256), 0, (hipStream_t)stream,
                     vox, nx, ny, nz, shift, cx, cy, f, out);
  return check_launch();
}

int launch_block_class(const uint2 *vox, int nx, int ny, int nz, int shift, const uint2 *cls,
                       const int2 *range, uint8_t *out, void *stream) {
  const int e = (1 << shift) - 1;
  const int bx = (nx + e) >> shift, by = (ny + e) >> shift, bz = (nz + e) >> shift;
  const int64_t nb = (int64_t)bx * by * bz;
  if (nb <= 0) return 0;
  hipLaunchKernelGGL(k_block_class, dim3(grid_for(nb, 256, 4096)), dim3(256), 0,
                     (hipStream_t)stream, vox, nx, ny, nz, shift, bx, by, nb, cls, range, out);
  return check_launch();
}

int launch_mh_fill(const float *f, int n_f, int C, uint64_t h_begin, uint64_t n, uint32_t key0,
                   uint32_t key1, int32_t *state, int32_t *out, void *stream) {
  if (C <= 0 || n == 0) return 0;
  hipLaunchKernelGGL(k_mh_fill, dim3((unsigned)((C + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, f, n_f, C, h_begin, n, key0, key1, state, out);
  return check_launch();
}

int launch_zero(void *ptr, size_t bytes, void *stream) {
  const size_t n = bytes / 8;
  if (n == 0) return 0;
  hipLaunchKernelGGL(k_zero, dim3(grid_for((int64_t)n, 256, 4096)), dim3(256), 0,
                     (hipStream_t)stream, (unsigned long long *)ptr, n);
  return check_launch();
}

int launch_sigma(const long long *s1, const unsigned long long *s2, const uint2 *vox, int64_t V,
                 uint32_t nb, double rho_min, double frac, int kind, double *scratch,
                 int nblocks, double *out, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  double *pmax = scratch;
  double *psum = scratch + nblocks;
  hipLaunchKernelGGL(k_sigma_max, dim3(nblocks), dim3(256), 0, s, s1, vox, V, rho_min, pmax);
  hipLaunchKernelGGL(k_sigma_sum, dim3(nblocks), dim3(256), 0, s, s1, s2, vox, V, nb, rho_min,
                     frac, kind, pmax, nblocks, psum);
  hipLaunchKernelGGL(k_sigma_final, dim3(1), dim3(256), 0, s, psum, nblocks, pmax, out);
  return check_launch();
}

int launch_read_dose(const long long *s1, const unsigned long long *s2, const uint2 *vox,
                     int64_t v0, int n, double vol, double n_hist, double per_batch, uint32_t nb,
                     double *out, void *stream) {
  hipLaunchKernelGGL(k_read_dose, dim3(grid_for(n, 256, 1024)), dim3(256), 0,
                     (hipStream_t)stream, s1, s2, vox, v0, n, vol, n_hist, per_batch, nb, out);
  return check_launch();
}

int launch_read_tally(const long long *s1, const unsigned long long *s2, int64_t v0, int n,
                      unsigned long long *out, void *stream) {
  hipLaunchKernelGGL(k_read_tally, dim3(grid_for(n, 256, 1024)), dim3(256), 0,
                     (hipStream_t)stream, (const unsigned long long *)s1, s2, v0, n, out);
  return check_launch();
}

int launch_microbench(int kind, void *buf_a, void *buf_b, int64_t n, int64_t ops, int grid,
                      void *stream) {
  hipStream_t s = (hipStream_t)stream;
  switch (kind) {
    case 0:
      hipLaunchKernelGGL(k_mb_copy, dim3(grid), dim3(256), 0, s, (const uint4 *)buf_a,
                         (uint4 *)buf_b, n / 16);
      break;
    case 1:
    case 2:
      hipLaunchKernelGGL(k_mb_atomic, dim3(grid), dim3(256), 0, s, (unsigned long long *)buf_a,
                         (uint32_t)(n / 8), kind == 2 ? 1 : 0, ops);
      break;
    case 3:
      hipLaunchKernelGGL(k_mb_gather, dim3(grid), dim3(256), 0, s, (const uint2 *)buf_a,
                         (uint32_t)(n / 8), ops, (uint32_t *)buf_b);
      break;
    default:
      return -1;
  }
  return check_launch();
}

int device_cu_count(int device) {
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) return 0;
  return prop.multiProcessorCount;
}

}  // namespace ctd
