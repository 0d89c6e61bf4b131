// k_sweep.hip -- the sweep launches of one plan (Sec. VIII.B): kernels that
// walk a job's tiles (sweep_tiles.h), tile choices, launch shapes, and the volumes'
// initial values.  k_sweep_batch.hip has the launches over many plans.
#include <atomic>

#include "sweep_tiles.h"

namespace nhp {
namespace {

// Workgroups stay resident and walk the tiles (the grid is capped near the
// number that fits the chip at once): a tile's stores drain while the next
// tile's loads are issued, and no workgroup launch separates them.  The
// barrier keeps the LDS tables of the previous tile until every wave is done
// with them.
template <int P, bool FUSED, bool GUARD, bool POW2>
__global__ __launch_bounds__(1024) void row_sweep_kernel(SweepJob job) {
  __shared__ RowShared sh;
  StepStore<P, false> none;
  StepKeep<P, false> keep(none);
  keep.set_geo(turn_geo<P, false>(job));
  for (int b = blockIdx.x; b < job.blocks; b += gridDim.x) {
    __syncthreads();
    row_sweep_tile<P, FUSED, GUARD, POW2, false>(job, tile_of(b, job.blocks, job.order), 0, sh, keep, -1);
  }
}

// The same with the tiles' stamps (SweepTrack): visits the active tiles only
// and stamps what their changes reach.
template <int P, bool FUSED, bool GUARD, bool POW2>
__global__ __launch_bounds__(1024) void row_track_kernel(SweepJob job) {
  constexpr bool LDS = steps_in_lds(P, true);
  __shared__ RowShared sh;
  __shared__ ActiveTiles at;
  __shared__ StepStore<P, LDS> store;
  StepKeep<P, LDS> keep(store);
  const TurnGeo geo = turn_geo<P, true>(job);  // (on its way while the active tiles are found)
  if (threadIdx.x == 0) sh.tr = job.tr;  // (read after the tiles' barriers)
  const bool skip = job.tr.mode == kTrackSkip;
  // with a workgroup per tile each looks at its own tile's stamp only
  const bool listed = skip && job.blocks > (int)gridDim.x;
  const int n = listed ? build_active(at, job) : job.blocks;
  keep.set_geo(geo);
  int swept = -1;  // tile whose changes are still to be stamped
  int parity = 0;
  for (int b = listed ? 0 : blockIdx.x; b < n; b += listed ? 1 : gridDim.x) {
    const int tile = listed ? __builtin_amdgcn_readfirstlane((int)at.list[b]) : tile_of(b, n, job.order);
    if (skip && !listed && tile_stamp(job, tile) <= job.tr.thr) continue;
    __syncthreads();
    row_sweep_tile<P, FUSED, GUARD, POW2, true>(job, tile, parity, sh, keep, swept);
    swept = tile;
    parity ^= 1;
  }
  if (swept >= 0) {
    __syncthreads();
    stamp_changes<P, FUSED, POW2>(job, swept, parity ^ 1, sh, keep);
  }
}

// Launch-shape knobs (nhp_set_knob; 0 = built-in choice).
std::atomic<int> g_knob[kKnobs];

}  // namespace

int knob(int k, int builtin) {
  const int v = g_knob[k].load(std::memory_order_relaxed);
  return v ? v : builtin;
}

// Resident workgroups for a row launch, on 256 CUs.
int row_grid(int blocks, int waves, int P) {
  const int cap = 256 * knob(NHP_KNOB_ROW_WG_PER_CU, row_workgroups(waves, P));
  return blocks < cap ? blocks : cap;
}

// Resident x-major workgroups: what fits a CU at once, times 256 CUs.
int xmajor_grid(int blocks, int per_cu) {
  const int cap = 256 * knob(NHP_KNOB_XMAJOR_WG_PER_CU, per_cu);
  return blocks < cap ? blocks : cap;
}

namespace {

template <int Q, int NT, int BUFS, bool TRACK>
__global__ __launch_bounds__(NT, (xband_waves_per_simd<Q, NT, BUFS>())) void xmajor_band_kernel(SweepJob job) {
  __shared__ XBand<Q, NT, BUFS> sh;
  for (int i = threadIdx.x; i < 2 * XBand<Q, NT, BUFS>::BROWS; i += NT) sh.dirty[i & 1][i >> 1] = 0;
  if (threadIdx.x < 2) sh.any[threadIdx.x] = 0;
  uint32_t chunks = 0;  // (the tile's first barrier orders the clearing before any flag is set)
  for (int b = blockIdx.x; b < job.blocks; b += gridDim.x) {
    const int tile = tile_of(b, job.blocks, job.order);
    if (TRACK && job.tr.mode == kTrackSkip && tile_stamp(job, tile) <= job.tr.thr) continue;
    xmajor_band_tile<Q, NT, BUFS, XBPREF, TRACK>(job, tile, sh, chunks);
  }
}

// (six transposed tiles of 27 KB fit a CU)
template <int Q, int NT, int BUFS>
__global__ __launch_bounds__(NT, 6) void xmajor_sweep_kernel(SweepJob job) {
  __shared__ XShared<Q, NT, BUFS> sh;
  for (int b = blockIdx.x; b < job.blocks; b += gridDim.x)
    xmajor_sweep_tile<Q, NT, BUFS>(job, tile_of(b, job.blocks, job.order), sh);
}

__device__ __forceinline__ void init_volume(const InitJob& j) {
  const size_t stride = (size_t)gridDim.x * blockDim.x, id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (size_t q = id; q < j.n_stamps; q += stride)
    j.stamps[q] = (q == j.marked[0] || q == j.marked[1] || q == j.marked[2]) ? 1u : 0u;
  for (size_t q = id; q < j.n4; q += stride) {
    const size_t e = q * 4;
    uint4 v = make_uint4(kInf, kInf, kInf, kInf);
    if (j.start >= e && j.start < e + 4) {
      const uint32_t o = (uint32_t)(j.start - e);
      if (o == 0) v.x = 0;
      if (o == 1) v.y = 0;
      if (o == 2) v.z = 0;
      if (o == 3) v.w = 0;
    }
    reinterpret_cast<uint4*>(j.V)[q] = v;
  }
}

__global__ void init_kernel(InitJob job) { init_volume(job); }

// Batched init: job k fills V of plan k; blocks stride over all plans' words.
__global__ void init_batch_kernel(const InitJob* __restrict__ jobs, int n_jobs) {
  for (int k = 0; k < n_jobs; k++) init_volume(jobs[k]);
}

__global__ void walls_kernel(uint8_t* __restrict__ B, int N, int L) {
  // one block per plane: row j = 0 and column i = 0 are hard
  const size_t base = (size_t)blockIdx.x * N * N;
  for (int k = threadIdx.x; k < N; k += blockDim.x) {
    B[base + k] = (uint8_t)kHard;
    B[base + (size_t)k * N] = (uint8_t)kHard;
  }
}

}  // namespace

// Whether the x-major kernel takes band tiles for grids of side N: a load
// round covers XBNT / (XBQ / 4) band rows, which must not exceed N (one wrap).
bool xmajor_wide(int N) { return N >= XBNT / (XBQ / 4); }

// Lines per x-major tile for grids of side N.
int xmajor_lines(int N) { return xmajor_wide(N) ? XBand<XBQ, XBNT, 1>::LINES : 64; }

// Steps per wave chosen for a curve length (0 = not set), process-wide.
static std::atomic<uint8_t> g_section_steps[1025];

int set_knob(int k, int v) {
  if (k < 0 || k >= kKnobs) return NHP_EINVAL;
  static const int lo[kKnobs] = {1, 1, 1, 1}, hi[kKnobs] = {8, 16, 2, 2};
  if (v != 0 && (v < lo[k] || v > hi[k])) return NHP_EINVAL;
  g_knob[k].store(v, std::memory_order_relaxed);
  return NHP_OK;
}

int get_knob(int k) { return (k < 0 || k >= kKnobs) ? -1 : g_knob[k].load(std::memory_order_relaxed); }

bool valid_section(int len, int P) { return (P == 8 || P == 16 || P == 32 || P == 64) && (len + P - 1) / P <= 16; }

// Steps per wave: the tuned choice for this curve length, else the smallest
// power of two in [8, 64] that splits the curve into at most 16 sections
// (16 waves of a 1024-thread workgroup).
int pick_section(int len) {
  if (len >= 1 && len <= 1024) {
    const int t = g_section_steps[len].load(std::memory_order_relaxed);
    if (t && valid_section(len, t)) return t;
  }
  int P = 8;
  while (P < 64 && P * 16 < len) P <<= 1;
  return (P * 16 >= len) ? P : 0;
}

int set_section_steps(int len, int P) {
  if (len < 1 || len > 1024) return NHP_EINVAL;
  if (P != 0 && !valid_section(len, P)) return NHP_EINVAL;
  g_section_steps[len].store((uint8_t)P, std::memory_order_relaxed);
  return NHP_OK;
}

void schedule_passes(const uint8_t* schedule, int n, uint64_t first, uint64_t count, bool pairs,
                     std::vector<Pass>& out) {
  const uint64_t end = first + count;
  for (uint64_t k = first; k < end;) {
    const int a = schedule[k % (uint64_t)n];
    if (pairs && k + 1 < end && fusable(a, schedule[(k + 1) % (uint64_t)n])) {
      out.push_back(Pass{(int8_t)a, (int8_t)schedule[(k + 1) % (uint64_t)n]});
      k += 2;
    } else {
      out.push_back(Pass{(int8_t)a, (int8_t)-1});
      k += 1;
    }
  }
}

bool can_fuse(const DevPlan& d) { return pick_section(d.nt) > 0; }

// The jobs of one pass of one plan: a row job (turns, or the y-major
// straight planes) and, for straights, an x-major job.  Returns the number of
// jobs written (0..2), blocks counts each job's workgroups; -1 for a pair
// that cannot share a pass (the caller splits it).
int make_sweep_jobs(const DevPlan& d, Pass pass, SweepJob* row, SweepJob* xmaj, TrackState* ts) {
  if (pass.mu2 >= 0 && !(fusable(pass.mu, pass.mu2) && can_fuse(d))) return -1;
  const int mu = pass.mu;
  const int N = d.nx, L = d.nt;
  const int tiles_x = (N + 63) / 64;
  SweepJob j{};
  j.V = d.V;
  j.B = d.B;
  j.N = N;
  j.n_poses = (uint32_t)N * (uint32_t)N * (uint32_t)L;
  j.ct = d.ct[mu];
  j.tiles_x = tiles_x;
  j.order = knob(NHP_KNOB_TILE_ORDER, 1);
  j.skew = d.skew;
  const StampLayout sl = stamp_layout(N, L);
  if (ts) {
    const uint32_t p = ++ts->pass;
    ts->sweeps += pass.mu2 >= 0 ? 2 : 1;
    // visit what changed since either maneuver's last pass
    uint32_t last = ts->last[mu];
    if (pass.mu2 >= 0 && last != kTrackStale) {
      const uint32_t other = ts->last[pass.mu2];
      if (other < last || other == kTrackStale) last = other;
    }
    j.tr.mode = last == kTrackStale ? kTrackAll : kTrackSkip;
    j.tr.thr = 2 * last;
    j.tr.mark_stamp = 2 * p;
    j.tr.own_stamp = pass.mu2 >= 0 ? 2 * p + 1 : 2 * p;
    j.tr.stamps = d.stamps;
    j.tr.turn_off = d.turn_off;
    j.tr.slot = d.slot;
    j.tr.nt = L;
    j.tr.n_planes_x = d.n_planes_x;
    ts->last[mu] = p;
    if (pass.mu2 >= 0) ts->last[pass.mu2] = p;
  }
  int n = 0;
  if (mu == NHP_SF || mu == NHP_SB) {
    j.L = N;
    j.cyclic = 0;
    j.edge_len = d.edge_len + (size_t)mu * L;
    j.fwd = d.fwd;
    j.mu_forward = (mu == NHP_SF);
    j.P = pick_section(N);
    SweepJob y = j, x = j;
    y.planes = d.planes + d.n_planes_x;
    y.blocks = tiles_x * d.n_planes_y;
    x.planes = d.planes;
    x.tiles_x = (N + xmajor_lines(N) - 1) / xmajor_lines(N);
    x.blocks = x.tiles_x * d.n_planes_x;
    x.P = 0;
    x.tr.own = (uint32_t)sl.str;
    y.tr.own = (uint32_t)sl.str + (uint32_t)d.n_planes_x;
    x.tr.pitch = y.tr.pitch = (uint32_t)L;
    row->blocks = 0;
    xmaj->blocks = 0;
    if (y.blocks) *row = y;
    if (x.blocks) *xmaj = x;
    n = (y.blocks > 0) + (x.blocks > 0);
  } else {
    const bool left = (mu == NHP_LF || mu == NHP_LB);
    j.L = L;
    j.cyclic = 1;
    j.dir = (mu == NHP_LF || mu == NHP_RB);  // eqs. (25)-(28): LF and RB step to T+1
    j.offx = d.turn_off + (left ? 0 : 2) * L;
    j.offy = d.turn_off + (left ? 1 : 3) * L;
    j.lq = d.turn_lq[mu];
    j.P = pick_section(L);
    if (pass.mu2 >= 0) {
      j.fused = 1;
      j.ct2 = d.ct[pass.mu2];
      j.lq2 = d.turn_lq[pass.mu2];
    }
    j.blocks = tiles_x * N;
    j.tr.own = (uint32_t)(left ? sl.left : sl.right);
    j.tr.pitch = (uint32_t)N;
    j.tr.circles = (uint32_t)(left ? sl.right : sl.left);
    j.tr.other_off = d.turn_off + (left ? 2 : 0) * L;
    *row = j;
    xmaj->blocks = 0;
    n = 1;
  }
  return n;
}

template <int P, bool FUSED, bool GUARD, bool POW2>
void launch_row_kernel(const SweepJob& j, hipStream_t s) {
  const int waves = (j.L + P - 1) / P;
  const dim3 grid(row_grid(j.blocks, waves, P)), block(64 * waves);
  if (j.tr.mode != kTrackOff)
    hipLaunchKernelGGL((row_track_kernel<P, FUSED, GUARD, POW2>), grid, block, 0, s, j);
  else
    hipLaunchKernelGGL((row_sweep_kernel<P, FUSED, GUARD, POW2>), grid, block, 0, s, j);
}

template <bool FUSED, bool GUARD, bool POW2>
hipError_t launch_row_job_t(const SweepJob& j, hipStream_t s) {
  switch (j.P) {
    case 64: launch_row_kernel<64, FUSED, GUARD, POW2>(j, s); break;
    case 32: launch_row_kernel<32, FUSED, GUARD, POW2>(j, s); break;
    case 16: launch_row_kernel<16, FUSED, GUARD, POW2>(j, s); break;
    case 8: launch_row_kernel<8, FUSED, GUARD, POW2>(j, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

bool is_pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }

template <bool FUSED, bool GUARD>
hipError_t launch_row_job_g(const SweepJob& j, hipStream_t s) {
  return is_pow2(j.N) ? launch_row_job_t<FUSED, GUARD, true>(j, s) : launch_row_job_t<FUSED, GUARD, false>(j, s);
}

hipError_t launch_row_job(const SweepJob& j, hipStream_t s) {
  const bool guard = j.L % j.P != 0;
  if (j.fused) return guard ? launch_row_job_g<true, true>(j, s) : launch_row_job_g<true, false>(j, s);
  return guard ? launch_row_job_g<false, true>(j, s) : launch_row_job_g<false, false>(j, s);
}

hipError_t launch_init(const DevPlan& d, uint32_t start_index, const StartTiles& marked, hipStream_t s) {
  InitJob j{};
  j.V = d.V;
  j.n4 = (size_t)d.nx * d.nx * d.nt / 4;  // a multiple of 16: nx and nt are multiples of 8
  j.start = start_index;
  j.stamps = d.stamps;
  j.n_stamps = (uint32_t)stamp_layout(d.nx, d.nt).words;
  for (int k = 0; k < 3; k++) j.marked[k] = marked.t[k];
  size_t blocks = (j.n4 + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(init_kernel, dim3((unsigned)blocks), dim3(256), 0, s, j);
  return hipGetLastError();
}

hipError_t launch_clear(uint32_t* words, size_t n, hipStream_t s) {
  InitJob j{};
  j.stamps = words;
  j.n_stamps = (uint32_t)n;
  for (uint32_t& m : j.marked) m = kNoTile;
  hipLaunchKernelGGL(init_kernel, dim3((j.n_stamps + 255) / 256), dim3(256), 0, s, j);
  return hipGetLastError();
}

hipError_t launch_init_batch(const InitJob* d_jobs, int n_jobs, size_t max_n4, hipStream_t s) {
  size_t blocks = (max_n4 + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(init_batch_kernel, dim3((unsigned)blocks), dim3(256), 0, s, d_jobs, n_jobs);
  return hipGetLastError();
}

hipError_t launch_force_walls(const DevPlan& d, hipStream_t s) {
  hipLaunchKernelGGL(walls_kernel, dim3(d.nt), dim3(256), 0, s, d.B, d.nx, d.nt);
  return hipGetLastError();
}

// Columns per chunk of a band launch.  A chunk costs the latency of its loads
// (one chunk ahead) and three barriers whatever its width, so a launch of at most
// two tiles per CU takes half as many chunks of 64 columns with 8 waves: 34 tiles
// (64^2 x 64) 8.1 -> 6.4 us, 152 (200^2 x 72) 18.3 -> 15.0, 396 (384^2 x 128) 33.8 -> 28.2.
// With more tiles than that the narrow chunks of several tiles per CU hide each
// other's latency.  Time of 64 columns over 32, passes that change nothing and passes
// that do, at 14 sides from 128 to 1024: 388 to 510 tiles 0.76-1.00 and 0.79-0.92
// (1000^2 x 56, 480 tiles: 89.9 -> 68.7 and 98 -> 79 us), 516 to 800 tiles 1.02-1.23
// and 1.02-1.14, but 0.93-1.03 and 1.04-1.05 at 1000^2.  (Chunks of 128 columns with 16 waves:
// 8.8, 16.0, 41.5 us and, at 520 tiles, 42.3 against 26.9.)  Shared launches, made for
// many plans, keep the narrow chunks.
constexpr int kFewBandTiles = 2 * 256;
bool wide_chunks(const SweepJob& j) { return j.N >= 64 && j.blocks <= kFewBandTiles; }

template <int Q, int NT, int BUFS>
void launch_band(const SweepJob& j, hipStream_t s) {
  const dim3 grid(xmajor_grid(j.blocks, kXBandGridPerCU)), block(NT);
  if (j.tr.mode != kTrackOff)
    hipLaunchKernelGGL((xmajor_band_kernel<Q, NT, BUFS, true>), grid, block, 0, s, j);
  else
    hipLaunchKernelGGL((xmajor_band_kernel<Q, NT, BUFS, false>), grid, block, 0, s, j);
}

bool trackable(const DevPlan& d) { return xmajor_wide(d.nx); }  // (transposed tiles keep no stamps)

hipError_t launch_sweep(const DevPlan& d, Pass pass, hipStream_t s, TrackState* ts) {
  return launch_sweep_part(d, pass, 3, s, ts);
}

hipError_t launch_sweep_part(const DevPlan& d, Pass pass, int parts, hipStream_t s, TrackState* ts) {
  SweepJob row{}, xmaj{};
  if (make_sweep_jobs(d, pass, &row, &xmaj, ts) < 0) {
    // a pair that cannot share a pass: one pass each
    const hipError_t e = launch_sweep(d, Pass{pass.mu, (int8_t)-1}, s, ts);
    return e != hipSuccess ? e : launch_sweep(d, Pass{pass.mu2, (int8_t)-1}, s, ts);
  }
  if (row.blocks && (parts & 1)) {
    if (!row.P) return hipErrorInvalidValue;
    const hipError_t e = launch_row_job(row, s);
    if (e != hipSuccess) return e;
  }
  if (xmaj.blocks && (parts & 2)) {
    const bool wide = xmajor_wide(xmaj.N);
    const bool one = knob(NHP_KNOB_XMAJOR_BUFFERS, wide ? XB_BUFS_BUILTIN : XBUFS_BUILTIN) == 1;
    if (wide) {
      if (one && wide_chunks(xmaj))
        launch_band<2 * XBQ, 2 * XBNT, 1>(xmaj, s);
      else if (one)
        launch_band<XBQ, XBNT, 1>(xmaj, s);
      else
        launch_band<XBQ, XBNT, 2>(xmaj, s);
    } else {
      const dim3 grid(xmajor_grid(xmaj.blocks, 6)), block(XNT);
      if (one)
        hipLaunchKernelGGL((xmajor_sweep_kernel<XQ, XNT, 1>), grid, block, 0, s, xmaj);
      else
        hipLaunchKernelGGL((xmajor_sweep_kernel<XQ, XNT, 2>), grid, block, 0, s, xmaj);
    }
    return hipGetLastError();
  }
  return hipSuccess;
}

}  // namespace nhp
