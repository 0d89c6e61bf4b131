// k_sweep_batch.hip -- batched sweep launches: the tiles of many plans' jobs
// (sweep_tiles.h) in one grid.
#include "sweep_tiles.h"

namespace nhp {
namespace {

// The tiles a tracked batched launch visits, as (tile, job): thread t looks at
// block t of the launch.  Tiles of a workgroup's 256 blocks stay together.
__global__ __launch_bounds__(256) void list_tiles_kernel(const SweepJob* __restrict__ jobs, int n_jobs,
                                                         int total_blocks, TileLists out) {
  __shared__ uint32_t count[4], at;
  const int t = blockIdx.x * 256 + threadIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = find_job(jobs, n_jobs, t < total_blocks ? t : total_blocks - 1);
  const SweepJob& a = jobs[j];
  const int tile = t - a.first_block;
  const bool on = t < total_blocks && (a.tr.mode != kTrackSkip || tile_stamp(a, tile) > a.tr.thr);
  const uint64_t m = __builtin_amdgcn_ballot_w64(on);
  if (lane == 0) count[wave] = (uint32_t)__builtin_popcountll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t n = count[0] + count[1] + count[2] + count[3];
    at = n ? atomicAdd(out.counters + out.which, n) : 0u;
    if (blockIdx.x == 0) out.counters[out.which ^ 1] = 0u;  // (its launch is over)
  }
  __syncthreads();
  uint32_t p = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  for (int w = 0; w < wave; w++) p += count[w];
  if (on && p < out.room) out.list[p] = make_uint2((uint32_t)tile, (uint32_t)j);
}

__device__ __forceinline__ int listed_tiles(const TileLists& in) {
  const uint32_t n = as_global((const uint32_t*)in.counters)[in.which];
  return __builtin_amdgcn_readfirstlane((int)umin(n, in.room));
}

// Listed tiles of a tracked batched launch (row_track_kernel over many jobs).
template <int P, bool FUSED, bool GUARD, bool POW2>
__global__ __launch_bounds__(1024) void row_track_batch_kernel(const SweepJob* __restrict__ jobs, TileLists in,
                                                                 int order) {
  constexpr bool LDS = steps_in_lds(P, true);
  __shared__ RowShared sh;
  __shared__ StepStore<P, LDS> store;
  StepKeep<P, LDS> keep(store);
  const int n = listed_tiles(in);
  int jg = -1;     // job whose tile was swept last, and whose geometry is kept
  int swept = -1;  // that tile, if its changes are still to be stamped
  int parity = 0;
  for (int b = blockIdx.x; b < n; b += gridDim.x) {
    __syncthreads();
    const uint2 e = in.list[tile_of(b, n, order)];
    const int tile = __builtin_amdgcn_readfirstlane((int)e.x), j = __builtin_amdgcn_readfirstlane((int)e.y);
    if (j != jg) {
      if (swept >= 0) {
        const SweepJob last = jobs[jg];
        stamp_changes<P, FUSED, POW2>(last, swept, parity ^ 1, sh, keep);
        swept = -1;
        __syncthreads();
      }
      keep.set_geo(turn_geo<P, true>(jobs[j]));
      if (threadIdx.x == 0) sh.tr = jobs[j].tr;  // (read after the tile's barriers)
      jg = j;
    }
    const SweepJob job = jobs[j];
    row_sweep_tile<P, FUSED, GUARD, POW2, true>(job, tile, parity, sh, keep, swept);
    swept = tile;
    parity ^= 1;
  }
  if (swept >= 0) {
    __syncthreads();
    const SweepJob last = jobs[jg];
    stamp_changes<P, FUSED, POW2>(last, swept, parity ^ 1, sh, keep);
  }
}

template <int P, bool FUSED, bool GUARD, bool POW2>
__global__ __launch_bounds__(1024) void row_sweep_batch_kernel(const SweepJob* __restrict__ jobs, int n_jobs,
                                                                 int total_blocks, int order) {
  __shared__ RowShared sh;
  int jg = -1;  // job whose turn geometry is kept
  StepStore<P, false> none;
  StepKeep<P, false> keep(none);
  for (int b = blockIdx.x; b < total_blocks; b += gridDim.x) {
    __syncthreads();
    const int t = tile_of(b, total_blocks, order);
    const int j = __builtin_amdgcn_readfirstlane(find_job(jobs, n_jobs, t));
    const SweepJob job = jobs[j];
    if (j != jg) {
      keep.set_geo(turn_geo<P, false>(job));
      jg = j;
    }
    row_sweep_tile<P, FUSED, GUARD, POW2, false>(job, t - job.first_block, 0, sh, keep, -1);
  }
}

template <int Q, int NT, int BUFS>
__global__ __launch_bounds__(NT, (xband_waves_per_simd<Q, NT, BUFS>())) void xmajor_band_batch_kernel(
    const SweepJob* __restrict__ jobs, int n_jobs, int order) {
  __shared__ XBand<Q, NT, BUFS> sh;
  const int t = tile_of(blockIdx.x, gridDim.x, order);
  const int j = __builtin_amdgcn_readfirstlane(find_job(jobs, n_jobs, t));
  const SweepJob job = jobs[j];
  for (int i = threadIdx.x; i < 2 * XBand<Q, NT, BUFS>::BROWS; i += NT) sh.dirty[i & 1][i >> 1] = 0;
  if (threadIdx.x < 2) sh.any[threadIdx.x] = 0;
  uint32_t chunks = 0;
  xmajor_band_tile<Q, NT, BUFS, XBPREF, false>(job, t - job.first_block, sh, chunks);
}

template <int Q, int NT, int BUFS>
__global__ __launch_bounds__(NT, (xband_waves_per_simd<Q, NT, BUFS>())) void xmajor_track_batch_kernel(
    const SweepJob* __restrict__ jobs, TileLists in, int order) {
  __shared__ XBand<Q, NT, BUFS> sh;
  const int n = listed_tiles(in);
  for (int i = threadIdx.x; i < 2 * XBand<Q, NT, BUFS>::BROWS; i += NT) sh.dirty[i & 1][i >> 1] = 0;
  if (threadIdx.x < 2) sh.any[threadIdx.x] = 0;
  uint32_t chunks = 0;
  for (int b = blockIdx.x; b < n; b += gridDim.x) {
    const uint2 e = in.list[tile_of(b, n, order)];
    const SweepJob job = jobs[__builtin_amdgcn_readfirstlane((int)e.y)];
    xmajor_band_tile<Q, NT, BUFS, XBPREF, true>(job, __builtin_amdgcn_readfirstlane((int)e.x), sh, chunks);
  }
}

template <int Q, int NT, int BUFS>
__global__ __launch_bounds__(NT, 6) void xmajor_sweep_batch_kernel(const SweepJob* __restrict__ jobs, int n_jobs,
                                                                  int order) {
  __shared__ XShared<Q, NT, BUFS> sh;
  const int t = tile_of(blockIdx.x, gridDim.x, order);
  const int j = __builtin_amdgcn_readfirstlane(find_job(jobs, n_jobs, t));
  const SweepJob job = jobs[j];
  xmajor_sweep_tile<Q, NT, BUFS>(job, t - job.first_block, sh);
}

}  // namespace

template <int P, bool FUSED, bool GUARD, bool POW2>
void launch_row_batch_kernel(const SweepJob* d_jobs, int n_jobs, int total_blocks, int waves, const TileLists* lists,
                             hipStream_t s) {
  const dim3 grid(row_grid(total_blocks, waves, P)), block(64 * waves);
  const int order = knob(NHP_KNOB_TILE_ORDER, 1);
  if (lists)
    hipLaunchKernelGGL((row_track_batch_kernel<P, FUSED, GUARD, POW2>), grid, block, 0, s, d_jobs, *lists, order);
  else
    hipLaunchKernelGGL((row_sweep_batch_kernel<P, FUSED, GUARD, POW2>), grid, block, 0, s, d_jobs, n_jobs,
                       total_blocks, order);
}

template <bool FUSED, bool GUARD, bool POW2>
hipError_t launch_row_batch_t(const SweepJob* d_jobs, int n_jobs, int total_blocks, int P, int waves,
                              const TileLists* l, hipStream_t s) {
  switch (P) {
    case 64: launch_row_batch_kernel<64, FUSED, GUARD, POW2>(d_jobs, n_jobs, total_blocks, waves, l, s); break;
    case 32: launch_row_batch_kernel<32, FUSED, GUARD, POW2>(d_jobs, n_jobs, total_blocks, waves, l, s); break;
    case 16: launch_row_batch_kernel<16, FUSED, GUARD, POW2>(d_jobs, n_jobs, total_blocks, waves, l, s); break;
    case 8: launch_row_batch_kernel<8, FUSED, GUARD, POW2>(d_jobs, n_jobs, total_blocks, waves, l, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <bool FUSED, bool GUARD>
hipError_t launch_row_batch_g(const SweepJob* d_jobs, int n_jobs, int total_blocks, int P, bool pow2, int waves,
                              const TileLists* l, hipStream_t s) {
  return pow2 ? launch_row_batch_t<FUSED, GUARD, true>(d_jobs, n_jobs, total_blocks, P, waves, l, s)
              : launch_row_batch_t<FUSED, GUARD, false>(d_jobs, n_jobs, total_blocks, P, waves, l, s);
}

hipError_t launch_sweep_batch(const SweepJob* d_jobs, int n_jobs, int total_blocks, int P, bool fused, bool guard,
                              bool pow2, bool xmajor, int waves, const TileLists* lists, hipStream_t s) {
  if (n_jobs == 0 || total_blocks == 0) return hipSuccess;
  if (lists) {
    hipLaunchKernelGGL(list_tiles_kernel, dim3((total_blocks + 255) / 256), dim3(256), 0, s, d_jobs, n_jobs,
                       total_blocks, *lists);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (xmajor) {
    const int order = knob(NHP_KNOB_TILE_ORDER, 1);
    const bool one = knob(NHP_KNOB_XMAJOR_BUFFERS, pow2 ? XB_BUFS_BUILTIN : XBUFS_BUILTIN) == 1;
    const dim3 grid(total_blocks);
    // (for x-major launches `pow2` says every job's grid takes band tiles)
    if (lists) {
      if (!pow2) return hipErrorInvalidValue;
      const dim3 walk(xmajor_grid(total_blocks, kXBandGridPerCU));
      if (one)
        hipLaunchKernelGGL((xmajor_track_batch_kernel<XBQ, XBNT, 1>), walk, dim3(XBNT), 0, s, d_jobs, *lists, order);
      else
        hipLaunchKernelGGL((xmajor_track_batch_kernel<XBQ, XBNT, 2>), walk, dim3(XBNT), 0, s, d_jobs, *lists, order);
      return hipGetLastError();
    }
    if (pow2 && one)
      hipLaunchKernelGGL((xmajor_band_batch_kernel<XBQ, XBNT, 1>), grid, dim3(XBNT), 0, s, d_jobs, n_jobs, order);
    if (pow2 && !one)
      hipLaunchKernelGGL((xmajor_band_batch_kernel<XBQ, XBNT, 2>), grid, dim3(XBNT), 0, s, d_jobs, n_jobs, order);
    if (!pow2 && one)
      hipLaunchKernelGGL((xmajor_sweep_batch_kernel<XQ, XNT, 1>), grid, dim3(XNT), 0, s, d_jobs, n_jobs, order);
    if (!pow2 && !one)
      hipLaunchKernelGGL((xmajor_sweep_batch_kernel<XQ, XNT, 2>), grid, dim3(XNT), 0, s, d_jobs, n_jobs, order);
    return hipGetLastError();
  }
  if (waves < 1 || waves > 16) return hipErrorInvalidValue;
  if (fused)
    return guard ? launch_row_batch_g<true, true>(d_jobs, n_jobs, total_blocks, P, pow2, waves, lists, s)
                 : launch_row_batch_g<true, false>(d_jobs, n_jobs, total_blocks, P, pow2, waves, lists, s);
  return guard ? launch_row_batch_g<false, true>(d_jobs, n_jobs, total_blocks, P, pow2, waves, lists, s)
               : launch_row_batch_g<false, false>(d_jobs, n_jobs, total_blocks, P, pow2, waves, lists, s);
}

}  // namespace nhp
