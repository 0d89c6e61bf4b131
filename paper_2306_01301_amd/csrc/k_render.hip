// k_render.hip -- obstacle rendering (Sec. VI) for gfx950, and soft
// obstacle costs from a distance transform of the image (Sec. VI-VII).
//
// For every heading plane T the obstacle volume is the maximum of the image
// codes under the vehicle box, taken separably: a sideways pass over the
// left-normal samples into a scratch plane, then a lengthwise pass over the
// heading samples.  The one-cell walls of Sec. V.C sit in row 0 and column 0
// of the image before dilation, and the wall poses themselves are forced
// hard afterwards.  Sample offsets come from the host (one table per plane).
// The image and a scratch plane stay L2-resident; the volume is written
// once.  The value volume's memory serves as the scratch volume.
#include <string.h>

#include "nhp_internal.h"

namespace nhp {
namespace {

// Sample offsets arrive reduced modulo N (in [0, N)), so one conditional
// subtraction wraps a row.
__device__ __forceinline__ int wrapn(int v, int N) { return v - ((v >= N) ? N : 0); }

__device__ __forceinline__ int tap_dx(int32_t p) { return (int)(p & 0xffff); }
__device__ __forceinline__ int tap_dy(int32_t p) { return (int)((uint32_t)p >> 16); }

// Both passes read rows that are padded to 2N columns (column x holds column
// x mod N), so a sample at column offset dx in [0, N) of pose column i is
// column i + dx of the padded row: no per-lane wrap.  The scratch space (the
// value volume, 4 bytes per pose) holds the padded sideways volume (2 bytes
// per pose) followed by the padded walled image (2 N^2 bytes).
__device__ __forceinline__ uint8_t* padded_image(const RenderJob& r) {
  return r.side + (size_t)2 * r.N * r.N * r.nt;
}

// A thread renders 4 W consecutive poses of a row (W words).  A sample's
// bytes at an arbitrary column come from W + 1 aligned words funnelled with one
// byte align per word, and the maximum runs on the bytes as two pairs of 16-bit
// lanes whose high bytes they are: the odd bytes as the word stands, the even
// ones shifted up by 8; the bytes below only break ties.  Sample offsets are the
// same for the whole block (one heading plane): staged in LDS, each is read
// into a scalar register.  Samples are taken 4 at a time with independent loads
// (the count is a run-time value).  The kernels are bound by the vector cache's
// data path and by this arithmetic, not by HBM, so more words per thread pay: 5
// words loaded for 4 words of poses against 2 for 1, and addresses worked out a
// quarter as often.  Lengthwise pass with 1 and with 4 words: 1010 -> 633 us at
// 1024^2 x 512 with 12 samples (1.6 GB moved: 0.31 ms at the copy rate), 186 ->
// 134 us at 256^2 x 256 with 90; sideways 505 -> 334 and 81 -> 60 us.  What is
// left is the vector cache: 56 cycles of a CU per sample and 1024 poses, 25 of
// them arithmetic.
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

template <int W>
struct __attribute__((packed, aligned(4))) WordRun {
  uint32_t w[W + 1];
};

template <int W>
__device__ __forceinline__ void max_over(const uint8_t* __restrict__ src, const int32_t* tp, int n, uint32_t i0, int j,
                                         int N, uint32_t (&out)[W]) {
  const uint32_t pitch = 2u * (uint32_t)N;  // a padded plane is below 2^21 bytes
  ushort2_t me[W], mo[W];
#pragma unroll
  for (int e = 0; e < W; e++) me[e] = mo[e] = ushort2_t{0, 0};
  auto load = [&](int32_t t) {
    // (i0 is a multiple of 4, so the words start at the sample's own alignment)
    const uint32_t at = __umul24((uint32_t)wrapn(j + tap_dy(t), N), pitch) + i0 + ((uint32_t)tap_dx(t) & ~3u);
    return *reinterpret_cast<const WordRun<W>*>(src + at);
  };
  auto take = [&](const WordRun<W>& q, int32_t t) {
#pragma unroll
    for (int e = 0; e < W; e++) {
      const uint32_t win = __builtin_amdgcn_alignbyte(q.w[e + 1], q.w[e], (uint32_t)t & 3u);
      mo[e] = __builtin_elementwise_max(mo[e], __builtin_bit_cast(ushort2_t, win));
      me[e] = __builtin_elementwise_max(me[e], __builtin_bit_cast(ushort2_t, win << 8));
    }
  };
  int g = 0;
  for (; g + 4 <= n; g += 4) {
    WordRun<W> q[4];
    int32_t t[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      t[e] = __builtin_amdgcn_readfirstlane(tp[g + e]);
      q[e] = load(t[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; e++) take(q[e], t[e]);
  }
  for (; g < n; g++) {
    const int32_t t = __builtin_amdgcn_readfirstlane(tp[g]);
    take(load(t), t);
  }
#pragma unroll
  for (int e = 0; e < W; e++)
    out[e] = (__builtin_bit_cast(uint32_t, mo[e]) & 0xFF00FF00u) | ((__builtin_bit_cast(uint32_t, me[e]) >> 8) & 0x00FF00FFu);
}

// One render job per plan; a block covers kRenderRows rows of one plane:
// block -> (plane, row group); its threads walk the rows' groups of 4 W poses.
constexpr int kRenderRows = 16;

__device__ __forceinline__ int find_render_job(const RenderJob* __restrict__ jobs, int n_jobs, int t) {
  int lo = 0, hi = n_jobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].first_block <= t)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Padded walled image, block b = row b: row 0 and column 0 (in both copies)
// are the walls of Sec. V.C.
__device__ __forceinline__ void pad_row(const RenderJob& r, int b) {
  const int N = r.N;
  uint8_t* P = padded_image(r) + (size_t)b * 2 * N;
  const uint8_t* src = r.image + (size_t)b * N;
  for (int x = threadIdx.x; x < 2 * N; x += blockDim.x) {
    const int xm = x < N ? x : x - N;
    P[x] = (b == 0 || xm == 0) ? (uint8_t)kHard : src[xm];
  }
}

// SIDE: side[T][j][i] = max over sideways samples of the walled image,
// written to both copies of the padded row.  Otherwise B[T][j][i] = max over
// lengthwise samples of side[T], walls forced hard.
template <bool SIDE, int W>
__device__ __forceinline__ void render_rows_w(const RenderJob& r, int b, const int32_t* tp) {
  const int N = r.N, G = N / (4 * W);
  const int groups = (N + kRenderRows - 1) / kRenderRows;
  const int T = b / groups, j0 = (b % groups) * kRenderRows;
  const int j1 = (j0 + kRenderRows) < N ? (j0 + kRenderRows) : N;
  const size_t NN = (size_t)N * N;
  const int n = SIDE ? r.n_side : r.n_len;
  const uint8_t* src = SIDE ? padded_image(r) : r.side + (size_t)T * 2 * NN;
  // the loop runs the same number of times in every lane, so the sample
  // offsets stay scalar loads (a lane past the end repeats the last group)
  const int total = (j1 - j0) * G;
  for (int base = 0; base < total; base += blockDim.x) {
    const int item = base + (int)threadIdx.x;
    const bool valid = item < total;
    const int it = valid ? item : total - 1;
    const int j = j0 + it / G;
    const uint32_t i0 = 4u * W * (uint32_t)(it % G);
    uint32_t m[W];
    max_over<W>(src, tp, n, i0, j, N, m);
    uint8_t* row = SIDE ? r.side + ((size_t)T * N + j) * 2 * N : r.B + (size_t)T * NN + (size_t)j * N;
    if (!SIDE) {
      if (i0 == 0) m[0] |= kHard;
#pragma unroll
      for (int e = 0; e < W; e++) m[e] = j == 0 ? 0xFFFFFFFFu : m[e];
    }
    if (valid) {
      uint32_t* dst = reinterpret_cast<uint32_t*>(row + i0);
#pragma unroll
      for (int e = 0; e < W; e++) dst[e] = m[e];
      if (SIDE) {
        dst = reinterpret_cast<uint32_t*>(row + i0 + N);
#pragma unroll
        for (int e = 0; e < W; e++) dst[e] = m[e];
      }
    }
  }
}

// Words per thread: as many as leave every thread of a block an item (16 rows
// of N poses) and divide the row.
template <bool SIDE>
__device__ __forceinline__ void render_rows(const RenderJob& r, int b, int32_t* tp) {
  const int N = r.N, groups = (N + kRenderRows - 1) / kRenderRows, T = b / groups;
  const int n = SIDE ? r.n_side : r.n_len;
  // the plane's sample offsets in LDS (global loads of them would be vector
  // loads: the stores below might alias them)
  const int32_t* tg = r.taps + (size_t)T * (r.n_side + r.n_len) + (SIDE ? 0 : r.n_side);
  for (int g = threadIdx.x; g < n; g += blockDim.x) tp[g] = tg[g];
  __syncthreads();
  if (N >= 256 && N % 16 == 0)
    render_rows_w<SIDE, 4>(r, b, tp);
  else if (N >= 128)
    render_rows_w<SIDE, 2>(r, b, tp);
  else
    render_rows_w<SIDE, 1>(r, b, tp);
}

__global__ __launch_bounds__(256) void pad_image_kernel(RenderJob r) { pad_row(r, blockIdx.x); }
__global__ __launch_bounds__(256) void render_side_kernel(RenderJob r) {
  __shared__ int32_t tp[kMaxTaps];
  render_rows<true>(r, blockIdx.x, tp);
}
__global__ __launch_bounds__(256) void render_len_kernel(RenderJob r) {
  __shared__ int32_t tp[kMaxTaps];
  render_rows<false>(r, blockIdx.x, tp);
}

// batched: the pad blocks of job k are N rows starting at pad_first (a
// running sum over the jobs); the pass blocks follow first_block
__global__ __launch_bounds__(256) void pad_image_batch_kernel(const RenderJob* __restrict__ jobs, int n_jobs) {
  int lo = 0, hi = n_jobs - 1, t = blockIdx.x;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].pad_first <= t)
      lo = mid;
    else
      hi = mid - 1;
  }
  pad_row(jobs[lo], t - jobs[lo].pad_first);
}

__global__ __launch_bounds__(256) void render_side_batch_kernel(const RenderJob* __restrict__ jobs, int n_jobs) {
  const int k = find_render_job(jobs, n_jobs, blockIdx.x);
  __shared__ int32_t tp[kMaxTaps];
  render_rows<true>(jobs[k], blockIdx.x - jobs[k].first_block, tp);
}

__global__ __launch_bounds__(256) void render_len_batch_kernel(const RenderJob* __restrict__ jobs, int n_jobs) {
  const int k = find_render_job(jobs, n_jobs, blockIdx.x);
  __shared__ int32_t tp[kMaxTaps];
  render_rows<false>(jobs[k], blockIdx.x - jobs[k].first_block, tp);
}

// ---- soft obstacle costs from a distance transform (Sec. VI-VII) ----
// Squared Euclidean distance to the nearest hard pixel, split the usual
// way: per column the squared distance to the nearest hard row, then per
// row the minimum over columns i' of (i - i')^2 + that column's value.  The
// table's last entry stands for every distance from len - 1 on, so neither
// search goes further than the radius whose square reaches len - 1.  Both
// kernels are bound by latency: 1024^2 pixels with a ramp of 24 cells take 3 +
// 14 us (386 + 93 us with whole columns per thread and whole rows per pixel),
// the call 30 us (832 us).

constexpr uint32_t kFar = 1u << 30;  // no hard pixel near enough in the column
constexpr int kMaxSoftRadius = 256;  // NHP_MAX_SOFT_TABLE entries

// A table that travels in the kernel's arguments (no copy of its own, which
// from pageable memory costs more than both kernels).
struct SoftTable {
  static constexpr int kBytes = 3072;
  uint8_t b[kBytes];
};

// Hard pixels as bits, 32 rows of a column in a word: thread (column, word).
// One block also lays the table down for the next kernel.  64-thread blocks:
// the longest chain is 32 loads, so the rows of a large image are spread over
// as many CUs as there are (1024^2: 386 us with a thread per whole column).
__global__ __launch_bounds__(64) void soft_bits_kernel(const uint8_t* __restrict__ image, uint32_t* __restrict__ bits,
                                                       int n, SoftTable t, int t_len, uint8_t* __restrict__ table) {
  const int i = blockIdx.x * 64 + threadIdx.x, w = blockIdx.y;
  if (blockIdx.x == 0 && w == 0)
    for (int k = threadIdx.x; k < t_len; k += 64) table[k] = t.b[k];
  if (i >= n) return;
  const uint8_t* col = image + (size_t)32 * w * n + i;
  const int rows = n - 32 * w < 32 ? n - 32 * w : 32;  // a multiple of 8
  uint32_t m = 0;
  for (int r0 = 0; r0 < rows; r0 += 8) {
#pragma unroll
    for (int r = 0; r < 8; r++) m |= (col[(size_t)(r0 + r) * n] == kHard ? 1u : 0u) << (r0 + r);
  }
  bits[(size_t)w * n + i] = m;
}

// One workgroup per row: the column distances of its pixels from the bit
// words above and below, in LDS between margins of kFar, then per pixel the
// columns outwards until no nearer pixel is possible.
__global__ __launch_bounds__(256) void soft_rows_kernel(const uint32_t* __restrict__ bits,
                                                        const uint8_t* __restrict__ table, uint32_t len,
                                                        uint8_t* __restrict__ out, int n, int radius) {
  __shared__ uint32_t row[1024 + 2 * kMaxSoftRadius];
  const int j = blockIdx.x, jw = j >> 5, jb = j & 31, words = (n + 31) >> 5;
  for (int x = threadIdx.x; x < radius; x += blockDim.x) row[x] = row[radius + n + x] = kFar;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    int d = radius;  // nearest hard row, at most `radius` away
    uint32_t m = bits[(size_t)jw * n + i];
    const uint32_t up = m << (31 - jb), down = m >> jb;
    if (up) d = __builtin_clz(up) < d ? __builtin_clz(up) : d;
    if (down) d = __builtin_ctz(down) < d ? __builtin_ctz(down) : d;
    for (int w = jw - 1; w >= 0 && j - (32 * w + 31) < d; w--) {
      m = bits[(size_t)w * n + i];
      if (m) {
        const int e = j - (32 * w + 31 - __builtin_clz(m));
        d = e < d ? e : d;
        break;
      }
    }
    for (int w = jw + 1; w < words && 32 * w - j < d; w++) {
      m = bits[(size_t)w * n + i];
      if (m) {
        const int e = 32 * w + __builtin_ctz(m) - j;
        d = e < d ? e : d;
        break;
      }
    }
    row[radius + i] = d < radius ? (uint32_t)(d * d) : kFar;
  }
  __syncthreads();
  for (int i0 = 0; i0 < n; i0 += blockDim.x) {  // (the same rounds in every lane)
    const int i = i0 + (int)threadIdx.x;
    const uint32_t* at = row + radius + (i < n ? i : n - 1);
    const uint32_t own = at[0];
    uint32_t best = own < len - 1 ? own : len - 1;
    for (int k = 1; __builtin_amdgcn_ballot_w64((uint32_t)(k * k) < best) != 0ull; k++) {
      const uint32_t a = at[-k], b = at[k];
      const uint32_t d = (uint32_t)(k * k) + (a < b ? a : b);
      best = d < best ? d : best;
    }
    // a hard pixel is the only one at distance 0 (of a table of one entry, whose
    // distances are not searched, the bit says so)
    if (i < n) {
      const bool hard = (bits[(size_t)jw * n + i] >> jb) & 1u;
      out[(size_t)j * n + i] = hard ? (uint8_t)kHard : table[best];
    }
  }
}

}  // namespace

bool soft_table_in_args(uint32_t len) { return len <= (uint32_t)SoftTable::kBytes; }

hipError_t launch_soft_costs(const uint8_t* image, uint32_t* bits_scratch, const uint8_t* h_table, uint8_t* d_table,
                             uint32_t len, uint8_t* out, int n, hipStream_t s) {
  int radius = 0;  // the smallest whose square reaches len - 1
  while ((uint32_t)(radius * radius) < len - 1) radius++;
  SoftTable t;
  int t_len = 0;
  if (soft_table_in_args(len)) {
    t_len = (int)len;
    memcpy(t.b, h_table, len);
  }
  hipLaunchKernelGGL(soft_bits_kernel, dim3((n + 63) / 64, (n + 31) / 32), dim3(64), 0, s, image, bits_scratch, n, t,
                     t_len, d_table);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(soft_rows_kernel, dim3(n), dim3(256), 0, s, bits_scratch, d_table, len, out, n, radius);
  return hipGetLastError();
}

int render_blocks(int N, int nt) { return ((N + kRenderRows - 1) / kRenderRows) * nt; }

hipError_t launch_render(const DevPlan& d, const uint8_t* image, int n_side, int n_len, hipStream_t s) {
  RenderJob r{};
  r.image = image;
  r.side = reinterpret_cast<uint8_t*>(d.V);  // 2 N_R bytes (padded rows), then the padded image: 2 N^2, of the 4 N_R-byte value volume
  r.B = d.B;
  r.taps = d.taps;
  r.N = d.nx;
  r.nt = d.nt;
  r.n_side = n_side;
  r.n_len = n_len;
  r.blocks = render_blocks(d.nx, d.nt);
  hipLaunchKernelGGL(pad_image_kernel, dim3(d.nx), dim3(256), 0, s, r);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(render_side_kernel, dim3(r.blocks), dim3(256), 0, s, r);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(render_len_kernel, dim3(r.blocks), dim3(256), 0, s, r);
  return hipGetLastError();
}

hipError_t launch_render_batch(const RenderJob* d_jobs, int n_jobs, int total_blocks, int total_pad_rows,
                               hipStream_t s) {
  if (n_jobs == 0) return hipSuccess;
  hipLaunchKernelGGL(pad_image_batch_kernel, dim3(total_pad_rows), dim3(256), 0, s, d_jobs, n_jobs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(render_side_batch_kernel, dim3(total_blocks), dim3(256), 0, s, d_jobs, n_jobs);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(render_len_batch_kernel, dim3(total_blocks), dim3(256), 0, s, d_jobs, n_jobs);
  return hipGetLastError();
}

}  // namespace nhp
