// sweep_tiles.h -- the tiles of the maneuver kernels (Sec. VIII.B, Insert 1) for gfx950.
//
// One maneuver kernel relaxes every pose once along the curves of one
// maneuver.  Per pose p in curve order, with u = V(p) and w = weight of the
// edge leaving p:
//     out = min(v, u)            stored to V(p)   (INF if p is hard)
//     v   = min(v, u + ct) + w   carried to the next pose
// Each pose is an affine min-plus map v -> min(v + D, C) with D = w and
// C = u + ct + w (a hard pose is (INF, INF), a reset), and these maps compose
// associatively: (D1, C1) then (D2, C2) = (D1 + D2, min(C1 + D2, C2)).  That
// is the section value / section distance pair of the paper's Sections
// technique (App. D, Inserts 3-5).  All additions saturate at INF.
//
// Work decomposition (one HBM read and one write per pose):
//   * a workgroup owns 64 curves (one per lane) over their full length;
//   * wave w of the S waves holds steps [wP, (w+1)P) of every curve in
//     registers (values, and the obstacle codes packed 4 per register);
//   * each wave composes its section into one (D, C) per curve, the S pairs
//     meet in LDS, and each wave derives the value entering its section:
//     for turns the fixed point of the cyclic composition (equal to the
//     paper's two loops around the circle), for straights the composition of
//     the sections before it, starting from INF at the wall;
//   * each wave replays its section from registers and stores.
// A unit of work is a job (one maneuver of one plan); a batched launch
// covers the tiles of many jobs, each block finding its job by a binary
// search over the jobs' first block.
// Turn curves and y-major straight lines put the 64 lanes on 64 consecutive
// x of one row, so every load and store is a contiguous row segment.  The
// x-major straight family (|tan| <= 1) puts the lanes on a column instead;
// those planes are loaded and stored row-wise into an LDS tile per wave and
// transposed there.
#pragma once

#include "nhp_internal.h"

// Structured buffer access to the sweep kernels' volumes: the record index is
// the pose index for both the 4-byte values and the 1-byte codes, so one
// per-lane index addresses both (the hardware applies the record size), and
// indices at or past the record count read 0 and drop stores instead of
// touching memory.  (The compiler's structured-buffer operations, declared
// by their intrinsic names.)
__device__ uint32_t buffer_load_u32(__amdgpu_buffer_rsrc_t r, uint32_t index, uint32_t voffset, uint32_t soffset,
                                    int aux) __asm("llvm.amdgcn.struct.ptr.buffer.load.i32");
__device__ uint8_t buffer_load_u8(__amdgpu_buffer_rsrc_t r, uint32_t index, uint32_t voffset, uint32_t soffset,
                                  int aux) __asm("llvm.amdgcn.struct.ptr.buffer.load.i8");
__device__ void buffer_store_u32(uint32_t v, __amdgpu_buffer_rsrc_t r, uint32_t index, uint32_t voffset,
                                 uint32_t soffset, int aux) __asm("llvm.amdgcn.struct.ptr.buffer.store.i32");

namespace nhp {
namespace {

__device__ __forceinline__ uint32_t sadd(uint32_t a, uint32_t b) { return __builtin_elementwise_add_sat(a, b); }
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

// Edge weight (Lq * (256 + 4 code) + 128) >> 8, infinite for a hard code.
// base = 256 Lq + 128, lq4 = 4 Lq (Lq <= 2^21 keeps the sum below 2^32).
__device__ __forceinline__ uint32_t weight(uint32_t code, uint32_t base, uint32_t lq4) {
  const uint32_t w = (base + lq4 * code) >> 8;
  return code == kHard ? kInf : w;
}

// A column in [0, 2N) reduced to [0, N): the unsigned i - N wraps above i
// whenever i < N, so the smaller of the two is the reduced column.
__device__ __forceinline__ uint32_t wrap_col(uint32_t i, int N) {
  const uint32_t j = i - (uint32_t)N;
  return j < i ? j : i;
}

// Index of the pose at column (x + shift) mod N of the row starting at pose
// rb (a multiple of N).  For a power-of-two N the geometry table holds
// g = rb | shift, and the pose is g + x with the carry out of the column
// bits dropped: the low bits of g + x spliced onto the high bits of g
// (one bitfield insert).
template <bool POW2>
__device__ __forceinline__ uint32_t row_cell(uint32_t g, uint32_t x, uint32_t shift, int N) {
  if (POW2) {
    const uint32_t m = (uint32_t)N - 1u;
    uint32_t r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "s"(m), "v"(g + x), "v"(g));  // (sum & m) | (g & ~m)
    return r;
  }
  return g + wrap_col(x + shift, N);
}

// bits |= any ? bit : 0 on scalar registers (any and bits are the same in all
// lanes; written out because the compiler folds such bits through vector
// registers, or keeps every mask live to the end).  A lone maneuver without
// stamps has the registers for it, and there the compiler's own order is the
// faster one (single turn 512^2 x 256: 67.0 us, written out 68.5): note_lone.
__device__ __forceinline__ void set_if(uint32_t& bits, uint32_t any, uint32_t bit) {
  uint32_t t;
  asm("s_cmp_lg_u32 %2, 0\n\ts_cselect_b32 %1, %3, 0\n\ts_or_b32 %0, %0, %1"
      : "+s"(bits), "=&s"(t)
      : "s"(any), "i"(bit)
      : "scc");
}

__device__ __forceinline__ void note_lone(uint32_t& bits, uint64_t mask, int k) {
  bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)(bits | ((mask != 0ull ? 1u : 0u) << k)));
}

constexpr int kBufferWord3 = 0x00020000;  // descriptor word 3 for untyped access on gfx9-family GPUs

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct RowBuffers {
  __amdgpu_buffer_rsrc_t V, B;
};
__device__ __forceinline__ RowBuffers row_buffers(const SweepJob& a) {
  return {__builtin_amdgcn_make_buffer_rsrc(a.V, (short)4, (int)a.n_poses, kBufferWord3),
          __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.B), (short)1, (int)a.n_poses, kBufferWord3)};
}

// A job's tables are global memory; saying so lets the compiler read them
// with global rather than generic loads (a job read from a batched job
// table otherwise reaches them through generic pointers).
template <typename T>
using GlobalPtr = __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ GlobalPtr<T> as_global(T* p) {
  return (GlobalPtr<T>)p;
}

// Workgroup index spread over the 8 XCDs so that consecutive tiles (which
// share row segments at their edges) land on the same XCD and its L2.
__device__ __forceinline__ int xcd_tile(int b, int n) {
  const int per = n >> 3, rem = n & 7, x = b & 7, k = b >> 3;
  return x * per + (x < rem ? x : rem) + k;
}

// Tile of workgroup slot b of n: XCD-aware (order 1) or launch order (order 2).
__device__ __forceinline__ int tile_of(int b, int n, int order) { return order == 2 ? b : xcd_tile(b, n); }

// ---- change tracking (SweepTrack) ----
// The x tiles that hold columns first .. first + w - 1 (cyclic; first in
// [0, N), w <= 66, w <= N); `tiles`: the stamp of x tile 0, `pitch` words per
// x tile.  Plain stores without a test for tiles stamped twice: lanes that
// stamp the same word share a request.
__device__ __forceinline__ void stamp_run(GlobalPtr<uint32_t> tiles, int pitch, int first, int w, int N, uint32_t stamp) {
  int mid = first + (w >> 1), last = first + w - 1;
  mid -= (mid >= N) ? N : 0;
  last -= (last >= N) ? N : 0;
  tiles[__umul24(first >> 6, pitch)] = stamp;
  if (w > 64) tiles[__umul24(mid >> 6, pitch)] = stamp;
  tiles[__umul24(last >> 6, pitch)] = stamp;
  // a short last tile may lie whole inside a run that wraps
  if ((N & 63) != 0 && last < first) tiles[__umul24((N - 1) >> 6, pitch)] = stamp;
}

__device__ __forceinline__ int below(int v, int N) { return v < 0 ? v + N : v; }  // v in [-N, N) reduced mod N

// The circle tiles (offsets ox, oy of their curves in this plane) that hold
// the run at columns col .. col + w - 1 of row `row`.
__device__ __forceinline__ void stamp_circles(GlobalPtr<uint32_t> st, int ox, int oy, int row, int col, int w, int N,
                                              uint32_t stamp) {
  stamp_run(st + below(row - oy, N), N, below(col - ox, N), w, N, stamp);
}

// The straight tiles of a plane (slope kq, straight_slope) that hold the run:
// lines x' = column - B(row) where lines advance a row per step, else x' =
// row - B(column) with B monotone.  B is taken from the slope, which is at
// most one off, so the run of lines is a line wider on both sides; reading
// the table instead would wait for every store still in flight.
__device__ __forceinline__ int slope_at(int kq, int y) { return (__mul24(y, kq) + 1024) >> 11; }
__device__ __forceinline__ void stamp_lines(GlobalPtr<uint32_t> st, int nt, int kq, bool x_major, int row, int col,
                                            int w, int N, uint32_t stamp) {
  const int end = col + w - 1;
  // the columns up to the end of the row (x-major: a wrapped rest starts another line run)
  const int b0 = (x_major && end >= N) ? N - 1 : end;
  const int ba = slope_at(kq, x_major ? col : row), bb = x_major ? slope_at(kq, b0) : ba;
  int x = (x_major ? row : col) - 1 - (ba > bb ? ba : bb);
  const int n = (x_major ? (ba > bb ? ba - bb : bb - ba) : w - 1) + 3;
  x = below(below(x, N), N);
  x -= (x >= N) ? N : 0;
  stamp_run(st, nt, x, n < N ? n : N, N, stamp);
  if (x_major && end >= N) {
    const int bc = slope_at(kq, end - N);
    int y = row - 1 - (bc > 0 ? bc : 0);
    const int m = (bc > 0 ? bc : -bc) + 3;
    y = below(y, N);
    y -= (y >= N) ? N : 0;
    stamp_run(st, nt, y, m < N ? m : N, N, stamp);
  }
}

// A plane's slope in 1/2048, from the last entry of its skew table.
__device__ __forceinline__ int straight_slope(int b_last, int N) {
  const int d = 2 * (N - 1), v = 2 * 2048 * b_last;
  const int k = (v + (v < 0 ? -(N - 1) : N - 1)) / d;
  return k > 2047 ? 2047 : (k < -2047 ? -2047 : k);
}

// Stamp of tile t of a job.
__device__ __forceinline__ GlobalPtr<uint32_t> own_stamp(const SweepJob& a, int t) {
  const int outer = t / a.tiles_x, tx = t - outer * a.tiles_x;
  return as_global(a.tr.stamps) + (a.tr.own + (uint32_t)tx * a.tr.pitch + (uint32_t)outer);
}
__device__ __forceinline__ uint32_t tile_stamp(const SweepJob& a, int t) { return *own_stamp(a, t); }

// The tiles a workgroup of a tracked launch visits when the launch has more
// tiles than workgroups.  Every workgroup reads the stamps of the job's tiles
// (at most 16384) once: a wave ballot gives 64 tiles' bits, a prefix sum of
// their counts the rank of every active tile, and ranks are dealt to the
// workgroups as tiles are in an untracked launch: a contiguous eighth of them
// to each XCD (order 1), round-robin over its workgroups.
struct ActiveTiles {
  static constexpr int kMaxTiles = 16384, kMinGrid = 256;
  uint64_t bits[kMaxTiles / 64];
  uint32_t before[kMaxTiles / 64];  // active tiles in the words before this one
  uint32_t total;
  uint16_t list[kMaxTiles / kMinGrid];
};

// Fills at.list with this workgroup's tiles and returns their number.
__device__ __forceinline__ int build_active(ActiveTiles& at, const SweepJob& a) {
  const int tiles = a.blocks, order = a.order;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int words = (tiles + 63) >> 6;
  constexpr int R = 4;  // words per round: their loads go out together
  for (int w0 = wave; w0 < words; w0 += R * waves) {
    uint32_t st[R];
#pragma unroll
    for (int e = 0; e < R; e++) {
      const int t = 64 * (w0 + e * waves) + lane;
      st[e] = tile_stamp(a, t < tiles ? t : tiles - 1);
    }
#pragma unroll
    for (int e = 0; e < R; e++) {
      const int w = w0 + e * waves, t = 64 * w + lane;
      const uint64_t m = __builtin_amdgcn_ballot_w64(t < tiles && st[e] > a.tr.thr);
      if (lane == 0 && w < words) at.bits[w] = m;
    }
  }
  __syncthreads();
  if (wave == 0) {
    uint32_t run = 0;
    for (int w0 = 0; w0 < words; w0 += 64) {
      const int w = w0 + lane;
      const uint32_t n = w < words ? (uint32_t)__builtin_popcountll(at.bits[w]) : 0u;
      uint32_t sum = n;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(sum, o, 64);
        if (lane >= o) sum += y;
      }
      if (w < words) at.before[w] = run + sum - n;
      run += __shfl(sum, 63, 64);
    }
    if (lane == 0) at.total = run;
  }
  __syncthreads();
  const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane((int)at.total);
  // this workgroup's ranks: first, first + step, ... below end
  uint32_t first = blockIdx.x, step = gridDim.x, end = total;
  if (order != 2) {
    const uint32_t x = blockIdx.x & 7u, per = total >> 3, rem = total & 7u;
    const uint32_t base = x * per + (x < rem ? x : rem);
    first = base + (blockIdx.x >> 3);
    step = (gridDim.x - x + 7u) >> 3;  // workgroups of this XCD
    end = base + per + (x < rem ? 1u : 0u);
  }
  for (int w = wave; w < words; w += waves) {
    const uint64_t m = at.bits[w];
    const uint32_t r = at.before[w] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if (((m >> lane) & 1u) && r >= first && r < end && (r - first) % step == 0)
      at.list[(r - first) / step] = (uint16_t)(64 * w + lane);
  }
  __syncthreads();
  return first < end ? (int)((end - first + step - 1u) / step) : 0;
}

// Value entering this wave's section: the cyclic fixed point (turns) or the
// composition of the earlier sections from INF (straights).  Sections are
// visited in increasing order (forward) or decreasing order (the second
// maneuver of a fused pair, which walks the curves backwards).
template <bool BACKWARD = false>
__device__ __forceinline__ uint32_t section_carry(const uint32_t (*aggD)[64], const uint32_t (*aggC)[64], int S,
                                                  int wave, int lane, bool cyclic) {
  uint32_t C = kInf;
  if (cyclic) {
    // once around, starting with this section and ending with the one before it
    int s = wave;
    for (int t = 0; t < S; t++) {
      C = umin(sadd(C, aggD[s][lane]), aggC[s][lane]);
      if (BACKWARD)
        s = (s == 0) ? S - 1 : s - 1;
      else
        s = (s + 1 == S) ? 0 : s + 1;
    }
  } else if (BACKWARD) {
    for (int s = S - 1; s > wave; s--) C = umin(sadd(C, aggD[s][lane]), aggC[s][lane]);
  } else {
    for (int s = 0; s < wave; s++) C = umin(sadd(C, aggD[s][lane]), aggC[s][lane]);
  }
  return C;
}

struct RowShared {
  uint32_t aggD[16][64];
  uint32_t aggC[16][64];
  uint32_t aggD2[16][64];  // second maneuver of a fused pair
  uint32_t aggC2[16][64];
  uint32_t wlut[256];      // edge weight by obstacle code (INF for hard)
  uint32_t wlut2[256];     // the same for the second maneuver
  uint32_t row_base[1024]; // per step: index of the first pose of the row it reads
                           // (power-of-two N: OR the column offset below)
  uint16_t shift[1024];    // per step: column offset of curve x' (reduced mod N)
  // tracked sweeps: per 32 steps, the steps with a changed value among the
  // tile's first and last 32 curves
  uint32_t changed[2][32];
  int line[2][5];          // straights, by tile parity: the plane's circle offsets (left x, y, right x, y), direction
  SweepTrack tr;
};

// The scan phases of one section held in registers, then its stores.
// GUARD: the curve length is not a multiple of P, so the last section has
// fewer than P real steps and the steps past the curve are skipped (without
// it every section is full and the loops carry no conditions).
// Write elision: a pass changes few poses once the search front has gone
// by (about 5 % of the poses and 11 % of the 128-byte lines per pass of a
// 512^3 maze plan), so a wave does not store a step whose 64 values are all
// unchanged (memory already holds them).  The test is per wave and step: a
// ballot in the replay, one bit per step, and a uniform branch at the store
// (no per-lane work; a step with any change stores all its lanes).
template <int P, bool FUSED, bool GUARD, bool POW2, bool TRACK>
__device__ __forceinline__ void scan_section(const SweepJob& a, const RowBuffers& buf, RowShared& sh,
                                             uint32_t (&u)[P], uint32_t (&code)[P], int n_real, int S, int wave,
                                             int lane, bool cyclic, bool active, int xp, int first, int N) {
  uint32_t packed[FUSED ? P / 4 : 1];
  // bit k: some value at step k changed (wave-uniform); tracked sweeps keep
  // the first and the last 32 lanes apart
  uint32_t lo = 0, hi = 0;
  auto note = [&](int k, uint32_t before, uint32_t after) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(after != before);
    if (TRACK) {
      set_if(lo, (uint32_t)m, 1u << k);
      set_if(hi, (uint32_t)(m >> 32), 1u << k);
    } else if (FUSED) {
      set_if(lo, (uint32_t)m | (uint32_t)(m >> 32), 1u << k);
    } else {
      note_lone(lo, m, k);
    }
  };
  static_assert(P <= 32, "one bit per step");
  {
    // weights replace the codes; compose the section into (D, C):
    // min(C + w, u + ct + w) = min(C, u + ct) + w (saturating add is monotone).
    // A fused pair keeps the codes, packed four to a register, for the
    // second maneuver's weights (packing after the loads have landed, so it
    // does not hold the loads back).
    uint32_t D = 0, C = kInf;
    if (FUSED) {
#pragma unroll
      for (int q = 0; q < P / 4; q++) {
        packed[q] = code[4 * q] | (code[4 * q + 1] << 8) | (code[4 * q + 2] << 16) | (code[4 * q + 3] << 24);
        asm volatile("" : "+v"(packed[q]));  // keep the packed form (not P live codes)
      }
    }
#pragma unroll
    for (int k = 0; k < P; k++) code[k] = sh.wlut[code[k]];
#pragma unroll
    for (int k = 0; k < P; k++) {
      if (!GUARD || k < n_real) {
        C = sadd(umin(C, sadd(u[k], a.ct)), code[k]);
        D = sadd(D, code[k]);
      }
    }
    sh.aggD[wave][lane] = D;
    sh.aggC[wave][lane] = C;
  }
  __syncthreads();
  {
    uint32_t v = section_carry(sh.aggD, sh.aggC, S, wave, lane, cyclic);
    // replay: a hard pose has weight INF, and w >> 31 (arithmetic) is then
    // all ones, which forces its output to INF (weights of other codes stay
    // below 2^24).  (In the first replay of a fused pair this changes no
    // result, but a hard pose would count as changed in every pass.)
#pragma unroll
    for (int k = 0; k < P; k++) {
      const uint32_t w = code[k];
      const uint32_t uu = u[k];
      u[k] = umin(v, uu) | (uint32_t)((int32_t)w >> 31);
      note(k, uu, u[k]);
      v = sadd(umin(v, sadd(uu, a.ct)), w);
    }
    if (FUSED) {
      // second maneuver: the steps of the section in reverse order, its
      // weights replacing the codes
      uint32_t D2 = 0, C2 = kInf;
#pragma unroll
      for (int k = P - 1; k >= 0; k--) {
        if (!GUARD || k < n_real) {
          code[k] = sh.wlut2[(packed[k >> 2] >> (8 * (k & 3))) & 0xffu];
          C2 = sadd(umin(C2, sadd(u[k], a.ct2)), code[k]);
          D2 = sadd(D2, code[k]);
        }
      }
      sh.aggD2[wave][lane] = D2;
      sh.aggC2[wave][lane] = C2;
    }
  }
  if (FUSED) {
    __syncthreads();
    uint32_t v = section_carry<true>(sh.aggD2, sh.aggC2, S, wave, lane, cyclic);
#pragma unroll
    for (int k = P - 1; k >= 0; k--) {
      if (!GUARD || k < n_real) {
        const uint32_t w = code[k];
        const uint32_t uu = u[k];
        u[k] = umin(v, uu) | (uint32_t)((int32_t)w >> 31);
        note(k, uu, u[k]);
        v = sadd(umin(v, sadd(uu, a.ct2)), w);
      }
    }
  }
  if (TRACK && lane == 0) {
    sh.changed[0][wave] = lo;
    sh.changed[1][wave] = hi;
  }
  const uint32_t changed = lo | hi;
  // recompute the pose of every step rather than keeping P of them live
  int xs = xp;
  asm volatile("" : "+v"(xs));
  if (active) {
#pragma unroll
    for (int k = 0; k < P; k++) {
      if ((!GUARD || k < n_real) && ((changed >> k) & 1u)) {
        buffer_store_u32(u[k], buf.V,
                         row_cell<POW2>(sh.row_base[first + k], (uint32_t)xs, POW2 ? 0u : sh.shift[first + k], N), 0,
                         0, 0);
      }
    }
  }
}

// Sections of 64 steps (curves of up to 1024 poses in 16 waves): the first
// 32 values of a section stay in registers and the other 32 in LDS (128 KB
// for 16 waves), the codes are packed four to a register as they arrive
// (loaded in groups of 16, so that few byte loads hold registers at once),
// and each use reads its weight from the LDS table.  The compiler barriers
// every 8 steps tie the table and LDS reads to the carried value, so only a
// few are live at once (holding all 64 values and weights would spill).
template <int P, bool FUSED, bool GUARD, bool POW2>
__device__ __forceinline__ void scan_section_wide(const SweepJob& a, const RowBuffers& buf, RowShared& sh, int n_real,
                                                  int S, int wave, int lane, bool cyclic, bool active, int xp,
                                                  int first, int L, int N) {
  constexpr int G = 16;      // codes per load group
  constexpr int H = P / 2;   // values kept in registers
  __shared__ uint32_t upper[16][P - H][64];
  // write elision, as in scan_section: bit k of changed[k / 32] says some
  // lane's value at step k changed (wave-uniform)
  uint32_t changed[2] = {};
  auto note = [&](int k, uint32_t before, uint32_t after) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(after != before);
    if (FUSED)
      set_if(changed[k >> 5], (uint32_t)m | (uint32_t)(m >> 32), 1u << (k & 31));
    else
      note_lone(changed[k >> 5], m, k & 31);
  };
  uint32_t (*hi)[64] = upper[wave];
  uint32_t u[H], packed[P / 4];
  const int xl = active ? xp : N - 1;
  {
    uint32_t uh[P - H];
#pragma unroll
    for (int k = 0; k < P; k++) {
      const int s = first + k;
      const uint32_t v =
          buffer_load_u32(buf.V, row_cell<POW2>(sh.row_base[s], (uint32_t)xl, POW2 ? 0u : sh.shift[s], N), 0, 0, 0);
      if (k < H)
        u[k] = v;
      else
        uh[k - H] = v;
    }
#pragma unroll
    for (int h = 0; h < P / G; h++) {
      asm volatile("" ::: "memory");
      int xg = xl;
      asm volatile("" : "+v"(xg));  // recompute the cells rather than keep P of them
      uint32_t c[G];
#pragma unroll
      for (int e = 0; e < G; e++) {
        const int k = h * G + e;
        const int s = first + k;
        c[e] = buffer_load_u8(buf.B, row_cell<POW2>(sh.row_base[s], (uint32_t)xg, POW2 ? 0u : sh.shift[s], N), 0, 0,
                              0);
      }
#pragma unroll
      for (int q = 0; q < G / 4; q++) {
        packed[h * (G / 4) + q] = c[4 * q] | (c[4 * q + 1] << 8) | (c[4 * q + 2] << 16) | (c[4 * q + 3] << 24);
        asm volatile("" : "+v"(packed[h * (G / 4) + q]));
      }
    }
#pragma unroll
    for (int k = 0; k < P - H; k++) hi[k][lane] = uh[k];  // a wave reads back only its own slots
  }
  auto weight_of = [&](int k) { return sh.wlut[(packed[k >> 2] >> (8 * (k & 3))) & 0xffu]; };
  {
    uint32_t D = 0, C = kInf;
#pragma unroll
    for (int k = 0; k < P; k++) {
      if ((k & 7) == 0) asm volatile("" : "+v"(C), "+v"(D)::"memory");
      // a step past the curve (GUARD) is the identity map: weight 0, value INF
      const bool real = !GUARD || k < n_real;
      const uint32_t w = real ? weight_of(k) : 0u;
      const uint32_t uk = real ? (k < H ? u[k] : hi[k - H][lane]) : kInf;
      C = sadd(umin(C, sadd(uk, a.ct)), w);
      D = sadd(D, w);
    }
    sh.aggD[wave][lane] = D;
    sh.aggC[wave][lane] = C;
  }
  __syncthreads();
  {
    // opaque: the replay recomputes u + ct and the weights rather than the
    // compiler keeping the compose phase's copies
#pragma unroll
    for (int q = 0; q < P / 4; q++) asm volatile("" : "+v"(packed[q]));
#pragma unroll
    for (int k = 0; k < H; k++) asm volatile("" : "+v"(u[k]));
    uint32_t v = section_carry(sh.aggD, sh.aggC, S, wave, lane, cyclic);
#pragma unroll
    for (int k = 0; k < P; k++) {
      if ((k & 7) == 0) asm volatile("" : "+v"(v)::"memory");
      const bool real = !GUARD || k < n_real;
      const uint32_t w = real ? weight_of(k) : 0u;
      const uint32_t uu = real ? (k < H ? u[k] : hi[k - H][lane]) : kInf;
      const uint32_t out = umin(v, uu) | (uint32_t)((int32_t)w >> 31);
      note(k, uu, out);
      if (k < H)
        u[k] = out;
      else
        hi[k - H][lane] = out;
      v = sadd(umin(v, sadd(uu, a.ct)), w);
    }
  }
  if (FUSED) {
    // second maneuver: the steps in reverse order with its own weights
    auto weight2_of = [&](int k) { return sh.wlut2[(packed[k >> 2] >> (8 * (k & 3))) & 0xffu]; };
    {
#pragma unroll
      for (int q = 0; q < P / 4; q++) asm volatile("" : "+v"(packed[q]));
      uint32_t D2 = 0, C2 = kInf;
#pragma unroll
      for (int k = P - 1; k >= 0; k--) {
        if ((k & 7) == 7) asm volatile("" : "+v"(C2), "+v"(D2)::"memory");
        const bool real = !GUARD || k < n_real;
        const uint32_t w = real ? weight2_of(k) : 0u;
        const uint32_t uk = real ? (k < H ? u[k] : hi[k - H][lane]) : kInf;
        C2 = sadd(umin(C2, sadd(uk, a.ct2)), w);
        D2 = sadd(D2, w);
      }
      sh.aggD2[wave][lane] = D2;
      sh.aggC2[wave][lane] = C2;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < P / 4; q++) asm volatile("" : "+v"(packed[q]));
#pragma unroll
    for (int k = 0; k < H; k++) asm volatile("" : "+v"(u[k]));
    uint32_t v = section_carry<true>(sh.aggD2, sh.aggC2, S, wave, lane, cyclic);
#pragma unroll
    for (int k = P - 1; k >= 0; k--) {
      if ((k & 7) == 7) asm volatile("" : "+v"(v)::"memory");
      const bool real = !GUARD || k < n_real;
      const uint32_t w = real ? weight2_of(k) : 0u;
      const uint32_t uu = real ? (k < H ? u[k] : hi[k - H][lane]) : kInf;
      const uint32_t out = umin(v, uu) | (uint32_t)((int32_t)w >> 31);
      note(k, uu, out);
      if (k < H)
        u[k] = out;
      else
        hi[k - H][lane] = out;
      v = sadd(umin(v, sadd(uu, a.ct2)), w);
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int m = 0; m < 2; m++) sh.changed[0][2 * wave + m] = sh.changed[1][2 * wave + m] = changed[m];
  }
  int xs = xp;
  asm volatile("" : "+v"(xs));
  if (active) {
#pragma unroll
    for (int k = 0; k < P; k++) {
      if ((k & 7) == 0) asm volatile("" ::: "memory");
      if ((!GUARD || k < n_real) && ((changed[k >> 5] >> (k & 31)) & 1u)) {
        buffer_store_u32(k < H ? u[k] : hi[k - H][lane], buf.V,
                         row_cell<POW2>(sh.row_base[first + k], (uint32_t)xs, POW2 ? 0u : sh.shift[first + k], N), 0,
                         0, 0);
      }
    }
  }
}

// A turn job's step geometry is the same in every tile of the job: the
// plane, column offset and row offset of step s = threadIdx.x (a workgroup of
// 64 S threads covers the S P steps, since P <= 64).  The kernels read it
// once per job, so a turn tile's set-up reads no global memory and its loads
// are issued while the previous tile's stores are still draining (a global
// read there would first wait for every earlier store).
struct TurnGeo {
  // shift (column offset of the curve through x' = 0); tracked sweeps, 10 bits
  // each: shift, row offset of that curve from y', column offset of the other
  // circles, and the top bit: the plane's straights are x-major
  uint32_t own;
  // row offset of the curve from y'; tracked sweeps: row offset of the other
  // circles and slot of the plane (10 bits each), slope of the plane
  // (straight_slope, 12 bits)
  uint32_t other;
};
// Without stamps the two words are the tables' own, so nothing waits for them
// before the first tile's set-up (packed there too, single turns took 0.3-0.5 us
// more per launch: 256^2 x 128 9.0 -> 9.4 us, 384^2 x 128 18.5 -> 20.3).
template <int P, bool TRACK>
__device__ __forceinline__ TurnGeo turn_geo(const SweepJob& a) {
  TurnGeo g{0u, 0u};
  const int L = a.L, N = a.N, s = threadIdx.x;
  if (a.cyclic && s < ((L + P - 1) / P) * P) {
    const int sc = s < L ? s : L - 1;  // steps past the curve repeat the last one
    const int T = a.dir ? sc : (L - 1 - sc);
    g.own = (uint32_t)as_global(a.offx)[T];
    g.other = (uint32_t)as_global(a.offy)[T];
    if constexpr (TRACK) {
      const GlobalPtr<const int32_t> o = as_global(a.tr.other_off);
      const int k = straight_slope(as_global(a.skew)[(size_t)T * N + N - 1], N);
      const uint32_t slot = (uint32_t)as_global(a.tr.slot)[T];
      g.own |= (g.other << 10) | ((uint32_t)o[T] << 20) | (slot < (uint32_t)a.tr.n_planes_x ? 1u << 31 : 0u);
      g.other = (uint32_t)o[L + T] | (slot << 10) | ((uint32_t)k << 20);
    }
  }
  return g;
}

// What thread s keeps of step s between tiles: the job's turn geometry and,
// for the stamps of straights, the column offset it had in the tile before.
// Tracked sweeps keep it in LDS (only its own thread touches an entry) where
// there is room: in registers it is spilled, and reading a spilled register
// back waits for every store in flight (fused turn pass of a 512^2 x 256 plan
// 145 against 138 us).  The 64-step sections leave no room, and do not spill.
constexpr bool steps_in_lds(int P, bool track) { return track && P <= 32; }
template <int P, bool LDS>
struct StepStore {};
template <int P>
struct StepStore<P, true> {
  static constexpr int kSteps = 16 * P;
  TurnGeo geo[kSteps];
  uint16_t shift[kSteps];
};

template <int P, bool LDS>
struct StepKeep {
  TurnGeo g{0u, 0u};
  int s = 0;
  __device__ __forceinline__ explicit StepKeep(StepStore<P, LDS>&) {}
  __device__ __forceinline__ void set_geo(TurnGeo v) { g = v; }
  __device__ __forceinline__ TurnGeo geo() const { return g; }
  __device__ __forceinline__ void set_shift(int v) { s = v; }
  __device__ __forceinline__ int shift() const { return s; }
};
template <int P>
struct StepKeep<P, true> {
  using Store = StepStore<P, true>;
  Store& st;
  __device__ __forceinline__ explicit StepKeep(Store& s) : st(s) {}
  __device__ __forceinline__ void set_geo(TurnGeo g) {
    if (threadIdx.x < Store::kSteps) st.geo[threadIdx.x] = g;
  }
  __device__ __forceinline__ TurnGeo geo() const { return st.geo[threadIdx.x % Store::kSteps]; }
  __device__ __forceinline__ void set_shift(int v) {
    if (threadIdx.x < Store::kSteps) st.shift[threadIdx.x] = (uint16_t)v;
  }
  __device__ __forceinline__ int shift() const { return st.shift[threadIdx.x % Store::kSteps]; }
};

// Stamps of the tiles that hold changed poses of the tile swept before:
// thread s looks at step s (a barrier after the sweep has written sh.changed,
// and another before the next sweep writes it).  Reads no global memory, so
// nothing here waits for stores in flight.
template <int P, bool FUSED, bool POW2>
__device__ __forceinline__ void stamp_changes(const SweepJob& a, int tile, int parity, const RowShared& sh,
                                              const StepKeep<P, steps_in_lds(P, true)>& keep) {
  int s = threadIdx.x;
  asm volatile("" : "+v"(s));  // nothing of this is worked out ahead and kept over the tile loop (registers)
  const int N = a.N, L = a.L;
  if (s >= L) return;
  const int word = (s / P) * (P > 32 ? 2 : 1) + ((s % P) >> 5), bit = (s % P) & 31;
  const bool lo = (sh.changed[0][word] >> bit) & 1u, hi = (sh.changed[1][word] >> bit) & 1u;
  if (!lo && !hi) return;
  const bool cyclic = FUSED || a.cyclic != 0;
  const SweepTrack& tr = sh.tr;
  const GlobalPtr<uint32_t> st = as_global(tr.stamps);
  const uint32_t stamp = tr.mark_stamp;
  const int tiles_x = a.tiles_x, per = tiles_x * N;
  const int outer = POW2 ? tile >> __builtin_ctz(tiles_x) : tile / tiles_x, tx = tile - outer * tiles_x;
  st[tr.own + (uint32_t)tx * tr.pitch + (uint32_t)outer] = tr.own_stamp;
  // the changed part of the tile's columns of this row
  const int c0 = 64 * tx + (lo ? 0 : 32), c1 = 64 * tx + (hi ? 64 : 32), w = (c1 < N ? c1 : N) - c0;
  if (w <= 0) return;
  if (cyclic) {
    const TurnGeo g = keep.geo();
    int row = outer + (int)((g.own >> 10) & 1023u), col = c0 + (int)(g.own & 1023u);
    row -= (row >= N) ? N : 0;
    col -= (col >= N) ? N : 0;
    stamp_circles(st + tr.circles, (int)((g.own >> 20) & 1023u), (int)(g.other & 1023u), row, col, w, N, stamp);
    stamp_lines(st + 2 * per + ((g.other >> 10) & 1023u), L, (int32_t)g.other >> 20, (g.own >> 31) != 0u, row, col, w, N,
                stamp);
  } else {
    const int* o = sh.line[parity];
    const int row = o[4] ? s : L - 1 - s;
    int col = c0 + keep.shift();
    col -= (col >= N) ? N : 0;
    stamp_circles(st, o[0], o[1], row, col, w, N, stamp);
    stamp_circles(st + per, o[2], o[3], row, col, w, N, stamp);
  }
}

// Row-coalesced sweep of one tile (64 curves) of a job: turns (cyclic) and
// y-major straights.
//   turns:     tile -> (x tile, y'); step k -> plane T_k, offsets (ox, oy)
//   straights: tile -> (x tile, plane slot); step k -> row c_k, column x' + B(c_k)
// FUSED (turns): after the first maneuver the second one, on the same curves
// in the opposite direction, runs on the values still held in registers, so
// the pair costs one read and one write per pose.
// The workgroup has exactly one wave per section (64 S threads: the
// launchers size it so); a workgroup of another size skips the tile.
// POW2: N is a power of two.  swept: the tile this workgroup swept before,
// whose changes are stamped once this tile's loads are on their way (-1:
// none).
template <int P, bool FUSED, bool GUARD, bool POW2, bool TRACK>
__device__ __forceinline__ void row_sweep_tile(const SweepJob& a, int tile, int parity, RowShared& sh,
                                               StepKeep<P, steps_in_lds(P, TRACK)>& keep, int swept) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int N = a.N, L = a.L;
  const bool cyclic = FUSED || a.cyclic != 0;
  const int S = (L + P - 1) / P;  // sections of this job
  if ((int)blockDim.x != 64 * S) return;  // uniform over the workgroup
  const int tx = tile % a.tiles_x;
  const int outer = tile / a.tiles_x;  // y' (turns) or plane slot (straights)
  const int xp = tx * 64 + lane;
  const bool active = xp < N;
  const RowBuffers buf = row_buffers(a);

  int T0 = 0;
  uint32_t Lq = a.lq;
  int dir = a.dir;
  GlobalPtr<const int16_t> sk = nullptr;
  if (!cyclic) {
    T0 = as_global(a.planes)[outer];
    Lq = as_global(a.edge_len)[T0];
    dir = (as_global(a.fwd)[T0] > 0) == (a.mu_forward != 0);
    sk = as_global(a.skew) + (size_t)T0 * N;
    if (TRACK && threadIdx.x < 4)
      sh.line[parity][threadIdx.x] = as_global(a.tr.turn_off)[(int)threadIdx.x * a.tr.nt + T0];
    if (TRACK && threadIdx.x == 0) sh.line[parity][4] = dir;
  }
  for (int c = threadIdx.x; c < 256; c += blockDim.x) {
    sh.wlut[c] = weight((uint32_t)c, 256u * Lq + 128u, 4u * Lq);
    if (FUSED) sh.wlut2[c] = weight((uint32_t)c, 256u * a.lq2 + 128u, 4u * a.lq2);
  }
  // Step s of a curve touches row `row` of plane T at column (x' + shift)
  // mod N: a row base shared by the 64 lanes plus a small per-lane column.
  // The geometry of all steps goes to LDS once per workgroup.
  // Steps past the curve (the last section's tail when L is not a multiple
  // of P) repeat the geometry of the last step, so loads need no clamp.
  // (one step per thread: S P <= 64 S threads)
  int shift = 0;
  if (const int s = threadIdx.x; s < S * P) {
    uint32_t Tn;
    int row;
    if (cyclic) {
      const TurnGeo g = keep.geo();
      const int sc = s < L ? s : L - 1;
      Tn = (uint32_t)(dir ? sc : (L - 1 - sc)) * (uint32_t)N;
      shift = (int)(TRACK ? g.own & 1023u : g.own);
      row = outer + (int)(TRACK ? (g.own >> 10) & 1023u : g.other);
      row -= (row >= N) ? N : 0;
    } else {
      Tn = (uint32_t)T0 * (uint32_t)N;
      const int sc = s < L ? s : L - 1;
      const int c = dir ? sc : (L - 1 - sc);
      shift = sk[c];
      shift += (shift < 0) ? N : 0;
      row = c;
    }
    const uint32_t rb = (Tn + (uint32_t)row) * (uint32_t)N;
    if (POW2) {
      sh.row_base[s] = rb | (uint32_t)shift;
    } else {
      sh.row_base[s] = rb;
      sh.shift[s] = (uint16_t)shift;
    }
  }
  __syncthreads();  // weight table and geometry ready

  // Sections are P steps; steps past the curve length (when S P > L) are
  // identity maps that touch no memory.
  const int n_real = (L - wave * P) < P ? (L - wave * P) : P;  // real steps of this wave
  const int first = wave * P;
  if constexpr (P >= 64) {
    if constexpr (TRACK) {
      if (swept >= 0) stamp_changes<P, FUSED, POW2>(a, swept, parity ^ 1, sh, keep);
      if (!cyclic) keep.set_shift(shift);
    }
    scan_section_wide<P, FUSED, GUARD, POW2>(a, buf, sh, n_real, S, wave, lane, cyclic, active, xp, first, L, N);
  } else {
    // Short sections stamp the tile before first (with their loads in registers
    // the stamps would cost them a resident wave per SIMD), 32-step ones while
    // their loads are on the way.
    if constexpr (TRACK && P < 32) {
      if (swept >= 0) stamp_changes<P, FUSED, POW2>(a, swept, parity ^ 1, sh, keep);
    }
    uint32_t u[P];
    uint32_t code[P];
    {
      // Load this wave's section of the 64 curves.  Lanes past the grid edge
      // read a valid cell, so the loads carry no branch; lanes are independent
      // curves, so an idle lane's values are never stored.
      const int xl = active ? xp : N - 1;
#pragma unroll
      for (int k = 0; k < P; k++) {
        // the geometry reads take constant offsets from one address (steps past
        // the curve have a copy of the last step's geometry)
        const int s = first + k;
        const uint32_t cell = row_cell<POW2>(sh.row_base[s], (uint32_t)xl, POW2 ? 0u : sh.shift[s], N);
        u[k] = buffer_load_u32(buf.V, cell, 0, 0, 0);
        code[k] = buffer_load_u8(buf.B, cell, 0, 0, 0);
      }
    }
    if constexpr (TRACK && P == 32) {
      if (swept >= 0) stamp_changes<P, FUSED, POW2>(a, swept, parity ^ 1, sh, keep);
    }
    if (TRACK && !FUSED && !cyclic)
      keep.set_shift(POW2 ? (int)(sh.row_base[threadIdx.x & 1023] & (uint32_t)(N - 1)) : (int)sh.shift[threadIdx.x & 1023]);
    scan_section<P, FUSED, GUARD, POW2, TRACK>(a, buf, sh, u, code, n_real, S, wave, lane, cyclic, active, xp, first, N);
  }
}

// x-major straights (|tan| <= 1): line x' visits (c, x' + B(c)), so lines
// that are neighbours in x' sit in different rows at every step and a lane
// per line would read a column.  A workgroup of NT / 64 waves owns 64 lines
// and walks them along c in chunks of Q columns.  Per chunk the cells owned
// by its lines form a sheared band of at most 64 + Q - 1 rows; they are read
// row by row (contiguous segments, each cell exactly once) and written to an
// LDS tile indexed by (line, column), the waves scan Q / NW columns each for
// all 64 lines (section composition in LDS, carry from the previous chunk),
// write the results back into the tile, and the band is stored row by row.
// A band cell that no line of the tile owns gets a record index past the
// end of the plane (its load reads nothing and its store is dropped) and an
// LDS slot in a spare row, so no lane branches.  The tile is double
// buffered, so a chunk's stores and the next chunk's loads need no barrier
// between them.
template <int Q, int NT, int BUFS>
struct XShared {
  static constexpr int LINES = 64;
  static constexpr int NW = NT / 64;    // waves
  static constexpr int PITCH = Q + 1;   // odd pitch: lanes reading one column of 64 lines hit 64 banks
  static constexpr int SLOTS = (LINES + 1) * PITCH;  // 64 lines and the spare row
  // codes: rows of Q bytes padded to an odd number of words, so the byte
  // reads of one column of 64 lines also fall in distinct banks
  static constexpr int PITCH_B = 4 * (Q / 4 + ((Q / 4) % 2 == 0 ? 1 : 0));
  static constexpr int SLOTS_B = (LINES + 1) * PITCH_B;
  uint32_t tV[BUFS][SLOTS];
  uint8_t tB[BUFS][SLOTS_B];
  uint32_t aggD[NW][64];
  uint32_t aggC[NW][64];
  uint32_t wlut[256];
  int16_t skew[1024];  // B(c, T) of this plane
};

template <int Q, int NT, int BUFS>
__device__ __forceinline__ void xmajor_sweep_tile(const SweepJob& a, int tile, XShared<Q, NT, BUFS>& sh) {
  using X = XShared<Q, NT, BUFS>;
  constexpr int LINES = X::LINES, PITCH = X::PITCH, PITCH_B = X::PITCH_B, NW = X::NW;
  static_assert((PITCH_B / 4) % 2 == 1 && PITCH_B % 4 == 0 && PITCH_B >= Q, "odd word pitch for the codes");
  constexpr int SUB = Q / NW;   // columns per wave
  constexpr int ROWS = NT / Q;  // band rows per load round (a column per thread)
  constexpr int ITER = (LINES + Q - 1 + ROWS - 1) / ROWS;
  static_assert(NT % Q == 0 && Q % NW == 0 && Q % 4 == 0, "Q must divide the thread count and split over the waves");
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int N = a.N;
  const uint32_t NN = (uint32_t)N * (uint32_t)N;
  const int x0 = (tile % a.tiles_x) * LINES;
  const int T = as_global(a.planes)[tile / a.tiles_x];
  // this plane's values and codes as record arrays indexed by row * N + column
  const __amdgpu_buffer_rsrc_t bV =
      __builtin_amdgcn_make_buffer_rsrc(a.V + (size_t)T * NN, (short)4, (int)NN, kBufferWord3);
  const __amdgpu_buffer_rsrc_t bB =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.B) + (size_t)T * NN, (short)1, (int)NN, kBufferWord3);
  const uint32_t Lq = as_global(a.edge_len)[T];
  for (int c = tid; c < 256; c += NT) sh.wlut[c] = weight((uint32_t)c, 256u * Lq + 128u, 4u * Lq);
  const int dir = (as_global(a.fwd)[T] > 0) == (a.mu_forward != 0);
  const GlobalPtr<const int16_t> skg = as_global(a.skew) + (size_t)T * N;
  for (int c = tid; c < N; c += NT) sh.skew[c] = skg[c];
  __syncthreads();
  const int16_t* sk = sh.skew;
  const int kk = tid % Q;  // column of this thread in the load/store phases
  const int r0 = tid / Q;  // first band row of this thread; rows r0 + it * ROWS
  const int t_lim = (N - x0) < LINES ? (N - x0) : LINES;  // lines of this tile inside the grid
  const uint32_t spare = LINES * PITCH + kk;               // LDS slot for cells no line owns
  const uint32_t spare_b = LINES * PITCH_B + kk;
  constexpr uint32_t kNoRecord = 0xFFFFFFFFu;

  uint32_t carry = kInf;  // value carried along line x0 + lane into the chunk
  int buf = 0;
  for (int k0 = 0; k0 < N; k0 += Q, buf = (BUFS == 2) ? (buf ^ 1) : 0) {
    uint32_t* tV = sh.tV[buf];
    uint8_t* tB = sh.tB[buf];
    const int nq = (N - k0) < Q ? (N - k0) : Q;
    const int c_first = dir ? k0 : (N - 1 - k0);
    const int c_last = dir ? (k0 + nq - 1) : (N - 1 - (k0 + nq - 1));
    const int b_first = sk[c_first], b_last = sk[c_last];
    const int bmin = b_first < b_last ? b_first : b_last;
    // grid row of band row 0, reduced mod N (|B| < N, so x0 + bmin is in (-N, 2N))
    int band0 = x0 + bmin;
    band0 += (band0 < 0) ? N : 0;
    band0 -= (band0 >= N) ? N : 0;
    const bool col_ok = kk < nq;
    const int my_c = dir ? (k0 + kk) : (N - 1 - (k0 + kk));
    const int my_b = sk[col_ok ? my_c : c_first];
    const uint32_t tl = col_ok ? (uint32_t)t_lim : 0u;
    int row = band0 + r0;
    row -= (row >= N) ? N : 0;
    const uint32_t rel0 = (uint32_t)row * (uint32_t)N + (uint32_t)(col_ok ? my_c : 0);
    const int t0 = r0 + bmin - my_b;

    // load the band: band row r holds line t = r + bmin - B(c) of column c
    uint32_t lv[ITER], lc[ITER];
    {
      uint32_t rel = rel0;
      int t = t0;
#pragma unroll
      for (int it = 0; it < ITER; it++) {
        const uint32_t idx = (uint32_t)t < tl ? rel : kNoRecord;
        lv[it] = buffer_load_u32(bV, idx, 0, 0, 0);
        lc[it] = buffer_load_u8(bB, idx, 0, 0, 0);
        t += ROWS;
        rel = wrap_col(rel + (uint32_t)(ROWS * N), (int)NN);  // ROWS rows down, wrapping around the plane
      }
    }
    {
      // the slots are recomputed rather than kept from the loads (registers)
      int t = t0;
      asm volatile("" : "+v"(t));
#pragma unroll
      for (int it = 0; it < ITER; it++) {
        const bool own = (uint32_t)t < tl;
        tV[own ? (uint32_t)(t * PITCH + kk) : spare] = lv[it];
        tB[own ? (uint32_t)(t * PITCH_B + kk) : spare_b] = (uint8_t)lc[it];
        t += ROWS;
      }
    }
    __syncthreads();

    // scan: wave w takes columns [w SUB, (w+1) SUB) of the chunk for all 64 lines
    const int line_slot = lane * PITCH + wave * SUB;
    const int line_slot_b = lane * PITCH_B + wave * SUB;
    uint32_t u[SUB], w[SUB];
#pragma unroll
    for (int q = 0; q < SUB; q++) {
      const bool ok = wave * SUB + q < nq;  // uniform
      u[q] = ok ? tV[line_slot + q] : kInf;
      w[q] = ok ? sh.wlut[tB[line_slot_b + q]] : 0u;
    }
    uint32_t D = 0, C = kInf;
#pragma unroll
    for (int q = 0; q < SUB; q++) {
      C = sadd(umin(C, sadd(u[q], a.ct)), w[q]);
      D = sadd(D, w[q]);
    }
    sh.aggD[wave][lane] = D;
    sh.aggC[wave][lane] = C;
    __syncthreads();
    uint32_t v = carry;
    for (int s = 0; s < wave; s++) v = umin(sadd(v, sh.aggD[s][lane]), sh.aggC[s][lane]);
#pragma unroll
    for (int q = 0; q < SUB; q++) {
      if (wave * SUB + q < nq) {
        tV[line_slot + q] = umin(v, u[q]) | (uint32_t)((int32_t)w[q] >> 31);
        v = sadd(umin(v, sadd(u[q], a.ct)), w[q]);
      }
    }
    for (int s = 0; s < NW; s++) carry = umin(sadd(carry, sh.aggD[s][lane]), sh.aggC[s][lane]);
    __syncthreads();

    // store the band back (cells no line owns have no record: dropped)
    {
      uint32_t rel = rel0;
      int t = t0;
      asm volatile("" : "+v"(t), "+v"(rel));
#pragma unroll
      for (int it = 0; it < ITER; it++) {
        const bool own = (uint32_t)t < tl;
        buffer_store_u32(tV[own ? (uint32_t)(t * PITCH + kk) : spare], bV, own ? rel : kNoRecord, 0, 0, 0);
        t += ROWS;
        rel = wrap_col(rel + (uint32_t)(ROWS * N), (int)NN);
      }
    }
    if (BUFS == 1) __syncthreads();  // every wave has read the tile before the next chunk writes it
  }
}

// x-major straights on grids of at least 32 cells: the same 64 lines and
// chunks of 32 columns, with the band kept in LDS in its memory layout (band
// row by band row) rather than transposed on the way in.  A thread moves 4
// adjacent columns of a band row (one 16-byte load of values, one 4-byte
// load of codes) into 4 consecutive LDS words and one code word, with no
// per-cell arithmetic; the scan reads line t's cell of column c at band row
// t + B(c) - bmin, an offset that is the same for every line of the column,
// so a column read is one address per lane plus a wave-uniform offset.
// Rows of 33 value words and 9 code words: the 64 lines of one column sit in
// consecutive band rows, which an odd pitch spreads over distinct banks.
// The stores read the band back the same way: one 16-byte store where the
// tile owns all 4 cells of a group, and one store of the owned run where it
// owns only some of them (a group of a band row can hold the last lines of
// this tile and the first of the next); band rows whose values did not change
// are not stored.  PREF: the next chunk's band is loaded into registers while
// the current one is scanned and stored, so each workgroup keeps loads in
// flight through its whole loop.
// What bounds a tile is less its bytes than the instructions and LDS waits
// between two loads, so a section that changes nothing writes nothing back to
// the band, and a chunk without a change has no store phase and no barrier
// after it; what the stores need beyond the band is found only there.  512^3,
// x-major half of a straight pass that changes nothing: 108 -> 89 us (62 us for
// the bytes at a copy's rate); in a maze's tracked passes 105 -> 93.5 us.
// A spilled vector register costs more than this gains: its reload waits for
// the prefetched band.

template <int Q_, int NT, int BUFS>
struct XBand {
  static constexpr int Q = Q_;                          // chunk columns
  static constexpr int NW = NT / 64;                    // waves
  static constexpr int SUB = 8;                         // columns a wave scans
  static constexpr int WPG = Q / SUB;                   // waves per group of 64 lines
  static constexpr int LINES = 64 * (NW / WPG);         // lines of a tile
  static constexpr int GW = Q / 4;                      // 4-column groups per band row
  static constexpr int ROWS = NT / GW;                  // band rows per load round
  static constexpr int BROWS = LINES + Q;               // band rows held (at least LINES + Q - 1)
  static constexpr int ITER = (BROWS + ROWS - 1) / ROWS;  // load rounds
  static constexpr int PV = Q + 1;                      // value words per band row (odd)
  static constexpr int PBW = Q / 4 + 1;                 // code words per band row (odd)
  uint32_t tV[BUFS][BROWS * PV];
  uint32_t tB[BUFS][BROWS * PBW];
  uint32_t aggD[NW][64];
  uint32_t aggC[NW][64];
  uint32_t wlut[256];
  alignas(16) int16_t skew[1024];  // B(c, T) of this plane (read 8 entries at a time)
  int16_t first_col[1024];         // first column c with |B(c) - B(0)| = i (B is monotone in unit steps)
  uint8_t dirty[2][BROWS];         // band rows holding a changed value, by chunk parity
  uint32_t any[2];                 // a band row does
  int off[4];                      // tracked sweeps: the plane's circle offsets (left x, y, right x, y)
};

// Where this thread's group of 4 columns sits in a chunk's band: record
// index of its first cell in band row r0, and the lines (relative to the
// tile) that own its outer cells in that row (one more per ROWS rows down).
struct BandGroup {
  uint32_t base;
  int lo, hi;  // smallest and largest owner: the owners of a group form a run of consecutive lines
  bool ok;     // the group lies inside the chunk's columns
};

// `chunks` counts the chunks this workgroup has swept (across tiles): its
// parity selects the band-row change flags of a chunk, which start cleared.
template <int Q_, int NT, int BUFS, bool PREF, bool TRACK>
__device__ __forceinline__ void xmajor_band_tile(const SweepJob& a, int tile, XBand<Q_, NT, BUFS>& sh,
                                                 uint32_t& chunks) {
  using X = XBand<Q_, NT, BUFS>;
  constexpr int Q = X::Q, LINES = X::LINES, NW = X::NW, GW = X::GW, ROWS = X::ROWS, ITER = X::ITER;
  constexpr int PV = X::PV, PBW = X::PBW, BROWS = X::BROWS, SUB = X::SUB, WPG = X::WPG;
  static_assert(BUFS == 1 || BUFS == 2, "one or two band buffers");
  static_assert(NT % GW == 0 && Q % SUB == 0 && NW % WPG == 0, "groups tile the threads; columns split over the waves");
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int csec = wave % WPG;            // this wave's column section of a chunk (SUB columns)
  const int gfirst = wave - csec;         // first wave of this wave's group of 64 lines
  const int line = (wave / WPG) * 64 + lane;  // the line this lane scans (relative to the tile)
  const int N = a.N;
  const uint32_t NN = (uint32_t)N * (uint32_t)N;
  const int x0 = (tile % a.tiles_x) * LINES;
  const int T = as_global(a.planes)[tile / a.tiles_x];
  // this plane's values and codes, addressed by byte offset
  const __amdgpu_buffer_rsrc_t rV =
      __builtin_amdgcn_make_buffer_rsrc(a.V + (size_t)T * NN, (short)0, (int)(NN * 4u), kBufferWord3);
  const __amdgpu_buffer_rsrc_t rB =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.B) + (size_t)T * NN, (short)0, (int)NN, kBufferWord3);
  const uint32_t Lq = as_global(a.edge_len)[T];
  for (int c = tid; c < 256; c += NT) sh.wlut[c] = weight((uint32_t)c, 256u * Lq + 128u, 4u * Lq);
  const int dir = (as_global(a.fwd)[T] > 0) == (a.mu_forward != 0);
  const GlobalPtr<const int16_t> skg = as_global(a.skew) + (size_t)T * N;
  if (TRACK && tid < 4) sh.off[tid] = as_global(a.tr.turn_off)[tid * a.tr.nt + T];
  const int b0 = skg[0];
  const bool incr = skg[N - 1] >= b0;  // B ascends with the column (else descends)
  for (int c = tid; c < N; c += NT) {
    const int b = skg[c];
    sh.skew[c] = (int16_t)b;
    if (c == 0 || b != skg[c - 1]) sh.first_col[b >= b0 ? b - b0 : b0 - b] = (int16_t)c;
  }
  __syncthreads();
  const int16_t* sk = sh.skew;
  const int gw = tid % GW;  // column group of this thread in the load and store phases
  const int r0 = tid / GW;  // first band row of this thread; rows r0 + it * ROWS
  const int gs = dir ? gw : GW - 1 - gw;  // the group's place in the band row (memory order)
  const int t_lim = (N - x0) < LINES ? (N - x0) : LINES;  // lines of this tile inside the grid
  constexpr uint32_t kNoOffset = 0xFFFFFFF0u;  // past the end of either plane: loads nothing

  // chunk k0 walks memory columns k0 .. k0 + nq - 1 (dir) or N - 1 - k0
  // down to N - k0 - nq; band row 0 is grid row x0 + bmin (mod N), where
  // bmin is the smallest B over the chunk (B is monotone: at one end)
  // grid row of band row 0: x0 + bmin reduced mod N (|B| < N, x0 < N)
  auto band_row0 = [&](int bmin) {
    int row = x0 + bmin;
    row += (row < 0) ? N : 0;
    return row - (row >= N ? N : 0);
  };
  // (and brange, the difference of B between the chunk's ends)
  auto chunk_bmin = [&](int k0, int nq, int& brange) {
    const int b_first = sk[dir ? k0 : (N - 1 - k0)];
    const int b_last = sk[dir ? (k0 + nq - 1) : (N - k0 - nq)];
    brange = __builtin_amdgcn_readfirstlane(b_first < b_last ? b_last - b_first : b_first - b_last);
    return __builtin_amdgcn_readfirstlane(b_first < b_last ? b_first : b_last);
  };
  auto group_of = [&](int k0, int nq, int bmin, BandGroup& g) {
    g.ok = 4 * gw < nq;
    const int cw = g.ok ? (dir ? (k0 + 4 * gw) : (N - 4 - k0 - 4 * gw)) : 0;
    const int row = band_row0(bmin) + r0;  // r0 < ROWS <= N: at most one wrap
    g.base = (uint32_t)(row - (row >= N ? N : 0)) * (uint32_t)N + (uint32_t)cw;
    const int t_0 = r0 + bmin - sk[cw], t_3 = r0 + bmin - sk[cw + 3];  // owners of the outer cells
    g.lo = t_0 < t_3 ? t_0 : t_3;
    g.hi = t_0 < t_3 ? t_3 : t_0;
  };
  // a group some line of the tile owns in band row r0 + it ROWS is loaded;
  // the others load nothing
  auto load_band = [&](const BandGroup& g, u32x4 (&lv)[ITER], uint32_t (&lc)[ITER]) {
    uint32_t base = g.base;
#pragma unroll
    for (int it = 0; it < ITER; it++) {
      if (BROWS % ROWS != 0 && r0 + it * ROWS >= BROWS) break;  // past the rows held (uniform per wave)
      const bool any = g.ok && g.hi + it * ROWS >= 0 && g.lo + it * ROWS < t_lim;
      lv[it] = __builtin_amdgcn_raw_buffer_load_b128(rV, any ? base * 4u : kNoOffset, 0, 0);
      lc[it] = __builtin_amdgcn_raw_buffer_load_b32(rB, any ? base : kNoOffset, 0, 0);
      base = wrap_col(base + (uint32_t)(ROWS * N), (int)NN);  // ROWS rows down, wrapping around the plane
    }
  };
  auto put_band = [&](int buf, const u32x4 (&lv)[ITER], const uint32_t (&lc)[ITER]) {
    uint32_t* dv = sh.tV[buf] + r0 * PV + 4 * gs;
    uint32_t* db = sh.tB[buf] + r0 * PBW + gs;
#pragma unroll
    for (int it = 0; it < ITER; it++) {
      if (BROWS % ROWS != 0 && r0 + it * ROWS >= BROWS) break;
#pragma unroll
      for (int m = 0; m < 4; m++) dv[it * ROWS * PV + m] = lv[it][m];
      db[it * ROWS * PBW] = lc[it];
    }
  };

  u32x4 lv[ITER];
  uint32_t lc[ITER];
  BandGroup g;
  int nq = N < Q ? N : Q;
  int brange;
  int bmin = chunk_bmin(0, nq, brange);
  group_of(0, nq, bmin, g);
  if (PREF) load_band(g, lv, lc);
  uint32_t carry = kInf;  // value carried along line x0 + line into the chunk
  int buf = 0;
  for (int k0 = 0; k0 < N; k0 += Q, buf = (BUFS == 2) ? (buf ^ 1) : 0) {
    if (!PREF) load_band(g, lv, lc);
    put_band(buf, lv, lc);
    // groups the tile owns in part (the last lines of this tile and the first
    // of the next, or the reverse, in one band row): a band row's owned cells
    // run between two columns, where B(c) - bmin passes the row (first line)
    // and the row minus t_lim (past the last line), and those lie inside the
    // chunk only for the first brange rows after band row 0 and after band row
    // t_lim.  One lane of the last waves per such (row, edge) finds the column
    // from the first-column table and, when it falls inside a group, writes that
    // group's owned cells after the whole groups are stored; the other waves
    // store whole groups only.  A launch of few wide tiles is as long as one
    // workgroup's chain of steps: there the search is done for every chunk, where
    // the scan hides it (200^2 x 72: 15.3 us with the search in the store phase,
    // 14.9 here); other launches are bound by instructions and search only
    // chunks that changed.
    int pg_slot = -1;       // LDS slot of the partial group's first cell (-1: none)
    int pg_rho = 0;         // its band row
    uint32_t pg_rec = 0;    // its record index
    uint32_t pg_own = 0;    // owned cells of the group, bit m for memory column gm + m
    auto find_partial = [&] {
      if (const int e = tid - (NT - 2 * Q); e >= 0) {  // (whole waves)
        const int r = e % Q;
        if (r < brange) {
          const bool last = e >= Q;
          const int rho = last ? t_lim + r : r;
          // |B - B(0)| at the first column past the edge, in memory order
          const int v = last ? (incr ? r + 1 + bmin - b0 : b0 - (r + bmin))
                             : (incr ? rho + bmin + 1 - b0 : b0 - (rho + bmin));
          const int cb = sh.first_col[v];
          if (cb & 3) {
            const int gm = cb & ~3;  // memory column of the group
            int row = band_row0(bmin) + rho;
            while (row >= N) row -= N;  // rho < BROWS: at most BROWS / N + 1 wraps
            pg_rec = (uint32_t)row * (uint32_t)N + (uint32_t)gm;
            pg_slot = rho * PV + (gm - (dir ? k0 : (N - k0 - Q)));
            pg_rho = rho;
            // the cells before cb are owned when ownership stops there (the
            // first line's edge with B ascending, the last line's with B
            // descending), else the cells from cb on
            const uint32_t before = (1u << (cb & 3)) - 1u;
            pg_own = (last != incr) ? before : (0xFu & ~before);
          }
        }
      }
    };
    if constexpr (WPG > 4) find_partial();
    BandGroup gn;
    int nq_n = 0, bmin_n = 0, brange_n = 0;
    if (PREF && k0 + Q < N) {
      nq_n = (N - k0 - Q) < Q ? (N - k0 - Q) : Q;
      bmin_n = chunk_bmin(k0 + Q, nq_n, brange_n);
      group_of(k0 + Q, nq_n, bmin_n, gn);
      load_band(gn, lv, lc);
    }
    __syncthreads();

    // scan: wave w takes chunk columns [w SUB, (w+1) SUB) for all 64 lines;
    // line `lane` at chunk column k is band row lane + B(c_k) - bmin.  A
    // chunk's column count is a multiple of 8 (so is N), so a wave's columns
    // are all inside the chunk or all past it (an identity section).
    const bool wok = csec * SUB < nq;  // uniform
    const uint32_t* tV = sh.tV[buf];
    const uint8_t* tB = reinterpret_cast<const uint8_t*>(sh.tB[buf]);
    // change flags: this chunk's set is clear (it was cleared during the
    // previous chunk); clear the other set for the next chunk (the previous
    // chunk's stores read it, and every wave finished them before the
    // barrier above)
    const int par = (int)(chunks & 1u);
    for (int i = tid; i < BROWS; i += NT) sh.dirty[par ^ 1][i] = 0;
    if (tid == 0) sh.any[par ^ 1] = 0;
    uint32_t u[SUB], w[SUB];
    int soff[SUB];  // wave-uniform part of each column's value slot
    int orow[SUB];  // band row of line 0 at each column (wave-uniform)
    if (wok) {
      // the wave's 8 columns are 8 consecutive entries of the skew table
      // (ascending when dir, else descending), 16-byte aligned: one read,
      // unpacked in scalar registers
      const int cs = dir ? (k0 + csec * SUB) : (N - SUB - k0 - csec * SUB);
      const uint4 s8 = *reinterpret_cast<const uint4*>(sk + cs);
      const uint32_t sw[4] = {(uint32_t)__builtin_amdgcn_readfirstlane((int)s8.x),
                              (uint32_t)__builtin_amdgcn_readfirstlane((int)s8.y),
                              (uint32_t)__builtin_amdgcn_readfirstlane((int)s8.z),
                              (uint32_t)__builtin_amdgcn_readfirstlane((int)s8.w)};
      int offb[SUB];
#pragma unroll
      for (int q = 0; q < SUB; q++) {
        const int k = csec * SUB + q;
        const int e = dir ? q : (SUB - 1 - q);
        const int o = (int)(int16_t)(sw[e >> 1] >> (16 * (e & 1))) - bmin;  // band row of line 0
        const int pos = dir ? k : (Q - 1 - k);                              // column in the band row
        soff[q] = o * PV + pos;
        orow[q] = o;
        offb[q] = line * (4 * PBW) + (o * (4 * PBW) + pos);
      }
      uint32_t code[SUB];
#pragma unroll
      for (int q = 0; q < SUB; q++) {
        u[q] = tV[line * PV + soff[q]];
        code[q] = tB[offb[q]];
      }
#pragma unroll
      for (int q = 0; q < SUB; q++) w[q] = sh.wlut[code[q]];
    } else {
#pragma unroll
      for (int q = 0; q < SUB; q++) {
        u[q] = kInf;
        w[q] = 0u;
        soff[q] = 0;
        orow[q] = 0;
      }
    }
    uint32_t D = 0, C = kInf;
#pragma unroll
    for (int q = 0; q < SUB; q++) {
      C = sadd(umin(C, sadd(u[q], a.ct)), w[q]);
      D = sadd(D, w[q]);
    }
    sh.aggD[wave][lane] = D;
    sh.aggC[wave][lane] = C;
    __syncthreads();
    // the value carried into this wave's section and out of the chunk, from all
    // of the group's sections (read together: one wait)
    uint32_t v = carry;
    {
      uint32_t sd[WPG], sc[WPG];
#pragma unroll
      for (int i = 0; i < WPG; i++) {
        sd[i] = sh.aggD[gfirst + i][lane];
        sc[i] = sh.aggC[gfirst + i][lane];
      }
#pragma unroll
      for (int i = 0; i < WPG; i++) {
        carry = umin(sadd(carry, sd[i]), sc[i]);
        if (i + 1 == csec) v = carry;
      }
    }
    // most sections change no value: only one that does writes its changed
    // cells back to the band and flags their rows
    uint32_t changed = 0;
    {
      uint32_t r = v;
#pragma unroll
      for (int q = 0; q < SUB; q++) {
        changed |= (umin(r, u[q]) | (uint32_t)((int32_t)w[q] >> 31)) ^ u[q];
        r = sadd(umin(r, sadd(u[q], a.ct)), w[q]);
      }
    }
    if (wok && __builtin_amdgcn_ballot_w64(changed != 0u) != 0ull) {
      uint32_t* tVw = sh.tV[buf];
      int lpv = line * PV;
      asm volatile("" : "+v"(lpv));  // the slots are found again rather than kept from the reads (registers)
#pragma unroll
      for (int q = 0; q < SUB; q++) {
        const uint32_t out = umin(v, u[q]) | (uint32_t)((int32_t)w[q] >> 31);
        if (out != u[q]) {
          tVw[lpv + soff[q]] = out;
          sh.dirty[par][line + orow[q]] = 1;
        }
        v = sadd(umin(v, sadd(u[q], a.ct)), w[q]);
      }
      sh.any[par] = 1;
    }
    __syncthreads();

    if (__builtin_amdgcn_readfirstlane((int)sh.any[par]) != 0) {  // (the same in every wave)
      if (TRACK && tid < BROWS && sh.dirty[par][tid]) {
        int row = band_row0(bmin) + tid;
        while (row >= N) row -= N;
        const int c0 = dir ? k0 : (N - k0 - nq);  // the chunk's first column in memory order
        const GlobalPtr<uint32_t> st = as_global(a.tr.stamps);
        stamp_circles(st, sh.off[0], sh.off[1], row, c0, nq, N, a.tr.mark_stamp);
        stamp_circles(st + a.tiles_x * N, sh.off[2], sh.off[3], row, c0, nq, N, a.tr.mark_stamp);
        *own_stamp(a, tile) = a.tr.own_stamp;
      }

      if constexpr (WPG <= 4) find_partial();
      // store the band: a group the tile owns whole in one 16-byte store, then
      // the owned cells of the partly owned groups found above; a band row
      // whose values all stayed as loaded is not stored (memory holds them)
      {
        uint32_t pv[4];
        if (pg_slot >= 0 && !sh.dirty[par][pg_rho]) pg_slot = -1;
        if (pg_slot >= 0) {
#pragma unroll
          for (int m = 0; m < 4; m++) pv[m] = sh.tV[buf][pg_slot + m];
        }
        int rs = r0;
        asm volatile("" : "+v"(rs));
        const uint32_t* sv = sh.tV[buf] + rs * PV + 4 * gs;
        uint32_t base = g.base;
#pragma unroll
        for (int it = 0; it < ITER; it++) {
          if (BROWS % ROWS != 0 && r0 + it * ROWS >= BROWS) break;
          u32x4 val;
#pragma unroll
          for (int m = 0; m < 4; m++) val[m] = sv[it * ROWS * PV + m];
          const bool all = g.ok && g.lo + it * ROWS >= 0 && g.hi + it * ROWS < t_lim;
          if (sh.dirty[par][r0 + it * ROWS]) __builtin_amdgcn_raw_buffer_store_b128(val, rV, all ? base * 4u : kNoOffset, 0, 0);
          base = wrap_col(base + (uint32_t)(ROWS * N), (int)NN);
        }
        if (pg_slot >= 0) {
          // the owned cells are a run of 1 to 3 at one end of the group: one
          // store of the run's length (each cell a separate memory request
          // costs more than the cells' bytes)
          const int m0 = __builtin_ctz(pg_own), len = __builtin_popcount(pg_own);
          const uint32_t off = (pg_rec + (uint32_t)m0) * 4u;
          const uint32_t a0 = m0 ? pv[1] : pv[0];
          const uint32_t a1 = m0 == 0 ? pv[1] : (m0 == 1 ? pv[2] : pv[3]);
          const uint32_t a2 = m0 ? pv[3] : pv[2];
          typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
          typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
          if (len == 1) __builtin_amdgcn_raw_buffer_store_b32(m0 == 3 ? pv[3] : (m0 == 2 ? pv[2] : a0), rV, off, 0, 0);
          if (len == 2) __builtin_amdgcn_raw_buffer_store_b64(u32x2{m0 ? pv[2] : pv[0], m0 ? pv[3] : pv[1]}, rV, off, 0, 0);
          if (len == 3) __builtin_amdgcn_raw_buffer_store_b96(u32x3{a0, a1, a2}, rV, off, 0, 0);
        }
      }
      // every wave has read the band before the next chunk writes it, and
      // the tables before the next tile does
      if (BUFS == 1 || k0 + Q >= N) __syncthreads();
    }
    chunks++;
    if (PREF) {
      g = gn;
      nq = nq_n;
      bmin = bmin_n;
      brange = brange_n;
    } else if (k0 + Q < N) {
      nq = (N - k0 - Q) < Q ? (N - k0 - Q) : Q;
      bmin = chunk_bmin(k0 + Q, nq, brange);
      group_of(k0 + Q, nq, bmin, g);
    }
  }
}

// The job a block of a batched launch works on: jobs are listed in order of
// their first block, so a binary search over `first_block` finds it.
__device__ __forceinline__ int find_job(const SweepJob* __restrict__ jobs, int n_jobs, int t) {
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

// x-major workgroups may walk several tiles.  A tile's stores read only the
// LDS band, and the next tile writes its band after the barrier that follows
// its weight and skew tables, so a wave still storing never sees it
// overwritten.  Grids of at least 32 cells take band tiles
// (xmajor_band_tile), smaller ones the transposed tile.  Occupancy asked of
// the register allocator: the waves per SIMD that the LDS allows.
constexpr int XBQ = 32;          // band tiles: chunk columns
constexpr int XBNT = 256;        // band tiles: workgroup threads
constexpr bool XBPREF = true;    // band tiles: load the next chunk while scanning this one
constexpr int kLdsBytes = 160 * 1024;

// Band tiles resident per CU: what the LDS allows, at most 20 waves.  More
// (the LDS allows 28 waves of 4-wave tiles with one buffer) gain no time and
// evict band rows that neighbouring tiles share from the L2 before both have
// read them: 1.15 times the algorithmic fetch at 6 or 7 tiles per CU against
// 1.04 at 5.
template <int Q, int NT, int BUFS>
constexpr int xband_wg_per_cu() {
  const int by_lds = kLdsBytes / (int)sizeof(XBand<Q, NT, BUFS>);
  const int by_waves = 20 / (NT / 64) > 0 ? 20 / (NT / 64) : 1;
  return by_lds < by_waves ? by_lds : by_waves;
}
template <int Q, int NT, int BUFS>
constexpr int xband_waves_per_simd() { return xband_wg_per_cu<Q, NT, BUFS>() * (NT / 64) / 4; }

// Band tile launches give each tile a workgroup of its own (up to 16 per CU
// in the grid, of which the occupancy above keeps 5 resident): the
// dispatcher hands the next tile to whichever CU frees a slot first, which
// evens out tiles of uneven cost better than a fixed round-robin over
// resident workgroups (2-5 % faster at 1024 sides, 0-3 % at 512).
constexpr int kXBandGridPerCU = 16;

// transposed x-major tiles (grids under 32 cells): chunks of 32 columns,
// 256 threads per workgroup
constexpr int XQ = 32;   // x-major chunk columns
constexpr int XNT = 256;  // x-major workgroup threads
constexpr int XBUFS_BUILTIN = 2;  // x-major tile buffers unless a knob says otherwise
constexpr int XB_BUFS_BUILTIN = 1;  // the same for band tiles

}  // namespace
}  // namespace nhp
