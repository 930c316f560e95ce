// Spatial compression of the dense table into boxes.
//
// Paper, Section 4.1 / Figure 2: every entry starts as a unit rectangle; equal
// adjacent rectangles are merged when their union fills its bounding box.  The
// decision and the volume-normalised cost are compressed separately.
//
// The merge is made canonical by fixing an axis order; along each axis in
// turn, boxes that agree in value and in their extent on every other axis are
// chained when one starts where the previous one ends.
//
// GPU formulation.
//   pass 0  (dense, first axis a0): lanes walk lines of cells along a0 and flag
//           the cells where the value changes (cells whose operands do not fit
//           their levels hold (INF, NONE) by construction and are not read: a
//           bit map from the fill says which cells those are).  Consecutive
//           lanes hold consecutive cells, so the flags of 64 cells are one
//           ballot = one word of a bit mask in table order; the same flags are
//           also kept line-major.  A prefix sum of the popcounts gives every
//           run (= box) its index in table order.
//   pass a  (on boxes): a box looks at the cell just past its end on axis a.
//           If that cell is the low corner of a live box of the same value and
//           the same extents on all other axes, the two are linked; heads of
//           chains then absorb their chain.  The low corner of a box is found
//           in O(1) through the bit mask and the prefix sums.  After the first
//           of these passes the live boxes move to dense arrays; the trailing
//           passes over the innermost bit axes are one kernel.
//   final   live boxes are compacted in index order = sorted by low corner.
#include <hip/hip_runtime.h>
#include "dev_params.h"
#include "compress.h"

namespace mrl {

// ---------------------------------------------------------------- value equality
// Normalised costs c1/vol1 and c2/vol2 where the volumes differ only by the
// factor s1 : s2 of one size axis.  Exact: 128-bit cross multiplication.
__device__ __forceinline__ bool norm_equal(uint64_t c1, uint32_t s1, uint64_t c2, uint32_t s2) {
  if (c1 == kInf || c2 == kInf) return c1 == c2;
  uint64_t a_lo = c1 * s2, a_hi = __umul64hi(c1, s2);
  uint64_t b_lo = c2 * s1, b_hi = __umul64hi(c2, s1);
  return a_lo == b_lo && a_hi == b_hi;
}

// ---------------------------------------------------------------- pass 0
constexpr uint32_t kCellWords = 8;         // 64-cell words a wave of the lane-per-cell kernels takes (a wave per word is mostly wave launch)

// A line = all cells sharing every coordinate but a0.  General form (any stride that is no multiple
// of 64): one lane per cell compares its value with the cell before it on the line; a wave covers one
// 64-cell word of the table-order masks and writes it whole (ballots: no atomics, no zeroing).
// The values are read once and the pass should be bound by that, but a lane's two divisions and the
// 128-bit products of the sizes took longer (41 M cells with memory bounds: 160 us, now 102; 410 MB take 79): the place on the line is
// divided once per wave and carried on from word to word, the bits that say which cells fit come as
// words the whole wave shares, shifted by the stride for the cells before, and an axis without sizes
// compares values as they are.
__global__ __launch_bounds__(256) void head_flags_kernel(Geo g, uint32_t a0,
                                                         const uint64_t* __restrict__ cost,
                                                         const uint16_t* __restrict__ arg,
                                                         const unsigned long long* __restrict__ fitmap,
                                                         const uint32_t* __restrict__ axis_sizes,
                                                         unsigned long long* __restrict__ maskD,
                                                         unsigned long long* __restrict__ maskC) {
  const uint32_t s0 = g.stride[a0], se = s0 * g.ext[a0], n_words = (g.n + 63u) / 64u, lane = threadIdx.x & 63u;
  const uint32_t word0 = __builtin_amdgcn_readfirstlane((blockIdx.x * 4u + (threadIdx.x >> 6)) * kCellWords);     // a wave takes kCellWords words
  if (word0 >= n_words) return;
  const uint32_t back = s0 >> 6, shift = s0 & 63u;               // shift > 0
  const uint32_t step = 64u % se;
  uint32_t r = (word0 * 64u + lane) % se;                        // from the start of the cells that share the axes before a0
#pragma unroll
  for (uint32_t w = 0; w < kCellWords; w++) {
    const uint32_t word = word0 + w, cell = word * 64u + lane;
    if (word >= n_words) break;
    const bool active = cell < g.n;
    const unsigned long long fits = fitmap[word];                // cells that cannot fit hold (INF, NONE): not read
    const unsigned long long pfits = (word >= back ? fitmap[word - back] << shift : 0ull) |
                                     (word > back ? fitmap[word - back - 1u] >> (64u - shift) : 0ull);
    bool hd = active, hc = active;
    if (active && r >= s0) {
      uint64_t c = kInf, pc = kInf;
      uint32_t a = kNone, pa = kNone;
      if ((fits >> lane) & 1ull) { c = cost[cell]; a = arg[cell]; }
      if ((pfits >> lane) & 1ull) { pc = cost[cell - s0]; pa = arg[cell - s0]; }
      hd = a != pa;
      if (axis_sizes) {
        const uint32_t j = r / s0;
        hc = !norm_equal(c, axis_sizes[j], pc, axis_sizes[j - 1u]);
      } else {
        hc = c != pc;
      }
    }
    r += step;
    r -= r >= se ? se : 0u;
    const unsigned long long bd = __ballot(hd), bc = __ballot(hc);
    if (lane == 0) {
      maskD[word] = bd;
      maskC[word] = bc;
    }
  }
}

// The same for lines whose stride is a multiple of 64 cells (every table with at least 64
// entries per shape): the 64 lanes of a wave then stand on 64 consecutive cells at every step, so
// one 64-bit word of the fit bit map covers the step and one ballot is one word of the mask.  A
// step's cells lie far from the previous step's, so every read is a trip to HBM; to have few of
// them wait for each other, the fit words of up to 64 steps are fetched by one gather (lane t
// holds step t's word), and the values of 8 steps are fetched together before they are compared.
constexpr int kHeadBatch = 8;
constexpr uint32_t kHeadSpread = 32;

__device__ __forceinline__ unsigned long long readlane64(unsigned long long v, uint32_t lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), (int)lane);
  return (unsigned long long)hi << 32 | lo;
}

__global__ __launch_bounds__(256) void head_flags_wave_kernel(Geo g, uint32_t a0,
                                                              const uint64_t* __restrict__ cost,
                                                              const uint16_t* __restrict__ arg,
                                                              const unsigned long long* __restrict__ fitmap,
                                                              const uint32_t* __restrict__ axis_sizes,
                                                              unsigned long long* __restrict__ maskD,
                                                              unsigned long long* __restrict__ maskC,
                                                              unsigned long long* __restrict__ lineD,
                                                              unsigned long long* __restrict__ lineC) {
  const uint32_t s0 = g.stride[a0], e0 = g.ext[a0];
  const uint32_t n_lines = g.n / e0;                  // a multiple of 64, as s0 is
  const uint32_t lane = threadIdx.x & 63u;
  // Workgroups that run at the same time work on kHeadSpread distant parts of the table (measured:
  // the pass is a quarter faster than with neighbours side by side); four consecutive workgroups
  // stay together, as their 16 waves fill whole 128-byte lines of the masks.  The grid is padded
  // to a multiple of 4 * kHeadSpread workgroups.
  const uint32_t nch = gridDim.x >> 2, ch = blockIdx.x >> 2;
  const uint32_t blk = ((ch % kHeadSpread) * (nch / kHeadSpread) + ch / kHeadSpread) << 2 | (blockIdx.x & 3u);
  const uint32_t q = blk * 256u + threadIdx.x, q0 = q - lane;
  if (q0 >= n_lines) return;                          // the whole wave
  const uint32_t hi0 = q0 / s0;
  const uint32_t base0 = hi0 * s0 * e0 + (q0 - hi0 * s0);      // lane 0's first cell: a multiple of 64
  uint64_t pc = 0; uint32_t pa = 0, ps = 1;
  // a chunk = up to 64 steps: lane t fetches the fit word of step j0 + t, and in the end stores
  // the two mask words of that step; a line's own flags of the chunk are one word per lane
  for (uint32_t j0 = 0; j0 < e0; j0 += 64) {
    const uint32_t jt = j0 + lane;
    const unsigned long long words = jt < e0 ? fitmap[(base0 + jt * s0) >> 6] : 0ull;
    const uint32_t sizes = (axis_sizes && jt < e0) ? axis_sizes[jt] : 1u;
    const uint32_t n_here = e0 - j0 < 64u ? e0 - j0 : 64u;
    unsigned long long od = 0, oc = 0, wd = 0, wc = 0;
    // steps [0, n_live) hold the cells that fit; past them every cell holds (INF, NONE), so that
    // only step n_live can still start a run
    const unsigned long long live = __ballot(words != 0);
    const uint32_t n_live = live ? 64u - (uint32_t)__builtin_clzll(live) : 0u;
    for (uint32_t u0 = 0; u0 < n_live; u0 += kHeadBatch) {
      uint64_t c[kHeadBatch];
      uint32_t a[kHeadBatch];
#pragma unroll
      for (int u = 0; u < kHeadBatch; u++) {
        const uint32_t t = u0 + u < n_live ? u0 + u : n_live - 1;
        const bool fits = (readlane64(words, t) >> lane) & 1ull;
        const uint32_t cell = base0 + lane + (j0 + t) * s0;
        c[u] = fits ? cost[cell] : kInf;
        a[u] = fits ? (uint32_t)arg[cell] : kNone;
      }
#pragma unroll
      for (int u = 0; u < kHeadBatch; u++) {
        if (u0 + u < n_live) {
          const uint32_t t = u0 + u, j = j0 + t;
          const uint32_t sz = (uint32_t)__builtin_amdgcn_readlane((int)sizes, (int)t);
          const bool hd = j == 0 || a[u] != pa;
          const bool hc = j == 0 || !norm_equal(c[u], sz, pc, ps);
          pc = c[u]; pa = a[u]; ps = sz;
          const unsigned long long bd = __ballot(hd), bc = __ballot(hc);
          if (lane == t) { od = bd; oc = bc; }
          wd |= (unsigned long long)hd << t;
          wc |= (unsigned long long)hc << t;
        }
      }
    }
    if (n_live < n_here) {
      const uint32_t t = n_live;
      const bool hd = j0 + t == 0 || pa != kNone, hc = j0 + t == 0 || pc != kInf;
      const unsigned long long bd = __ballot(hd), bc = __ballot(hc);
      if (lane == t) { od = bd; oc = bc; }
      wd |= (unsigned long long)hd << t;
      wc |= (unsigned long long)hc << t;
      pc = kInf; pa = kNone;
      ps = (uint32_t)__builtin_amdgcn_readlane((int)sizes, (int)(n_here - 1));
    }
    if (jt < e0) {
      const uint32_t w = (base0 + jt * s0) >> 6;
      maskD[w] = od;
      maskC[w] = oc;
    }
    lineD[(size_t)(j0 >> 6) * n_lines + q] = wd;
    lineC[(size_t)(j0 >> 6) * n_lines + q] = wc;
  }
}

// alive[b]: 0 once box b has been merged into another; else kLive | the stamp of the last pass in
// which a box linked to it (one byte for both: a live box stays live when it is linked to, so the
// linking thread can store the whole byte, and a byte less per box is written when the boxes are made).
constexpr uint8_t kLive = 0x80;

// ---------------------------------------------------------------- prefix sums
// Items come in pairs: one wide load each, coalesced over a wave (both arrays start on 256 bytes
// and pairs on even items).
struct LoadPopc {
  const unsigned long long* p;
  __device__ __forceinline__ uint32_t one(uint32_t i) const { return (uint32_t)__popcll(p[i]); }
  __device__ __forceinline__ void two(uint32_t i, uint32_t& x, uint32_t& y) const {
    const ulonglong2 v = *(const ulonglong2*)(p + i);
    x = (uint32_t)__popcll(v.x);
    y = (uint32_t)__popcll(v.y);
  }
};
struct LoadFlag {
  const uint8_t* p;
  __device__ __forceinline__ uint32_t one(uint32_t i) const { return p[i] ? 1u : 0u; }
  __device__ __forceinline__ void two(uint32_t i, uint32_t& x, uint32_t& y) const {
    const uint32_t v = *(const uint16_t*)(p + i);
    x = v & 0xFFu ? 1u : 0u;
    y = v >> 8 ? 1u : 0u;
  }
};

// A tile is 2048 items of a workgroup of four waves; a wave has 512 consecutive ones in four rows of
// 128, two per lane and row.  A row adds up to at most 128 * 64, so two rows share a word.
// Bound by the number of memory requests: with eight items in a row per lane, read one by one, and the
// top in steps of 256 sums, the scans of a solved pipeline (7 M words, 12 M flags and the two smaller
// tables) took 484 us of kernel time, now 289 (apply over 7 M words 68 -> 25 us, the top 23 -> 9); the
// solve 5422 -> 5332 us, the smallest one 519 -> 488 us (four to eight launches fewer).
constexpr uint32_t kScanRows = 4, kScanRow = 128, kScanTile = 4 * kScanRows * kScanRow;
static_assert(kScanTile == kScanTileItems, "the caller's scratch is sized by the tile");
constexpr uint32_t kScanTop = 2048;         // more tiles than this are added up by scan_top_kernel

template <class L>
__device__ __forceinline__ void scan_load(const L& load, uint32_t first, uint32_t n, uint32_t (&x)[kScanRows], uint32_t (&y)[kScanRows]) {
#pragma unroll
  for (uint32_t r = 0; r < kScanRows; r++) {
    const uint32_t i = first + r * kScanRow;
    x[r] = y[r] = 0;
    if (i + 1 < n) load.two(i, x[r], y[r]);
    else if (i < n) x[r] = load.one(i);
  }
}

__device__ __forceinline__ uint32_t scan_first() {
  return blockIdx.x * kScanTile + (threadIdx.x >> 6) * (kScanRows * kScanRow) + (threadIdx.x & 63u) * 2;
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(v, d, 64);
    if ((int)(threadIdx.x & 63u) >= d) v += o;
  }
  return v;
}

__device__ __forceinline__ uint32_t block_reduce_256(uint32_t v, uint32_t* sh) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_down(v, d, 64);
  if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t t = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return t;
}

template <class L>
__global__ __launch_bounds__(256) void scan_tile_sums_kernel(L load, uint32_t n, uint32_t* __restrict__ tile_sum) {
  __shared__ uint32_t sh[4];
  uint32_t x[kScanRows], y[kScanRows], s = 0;
  scan_load(load, scan_first(), n, x, y);
#pragma unroll
  for (uint32_t r = 0; r < kScanRows; r++) s += x[r] + y[r];
  const uint32_t t = block_reduce_256(s, sh);
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = t;
}

// One workgroup: exclusive scan of tile_sum in place, 4096 sums at a time.
__global__ __launch_bounds__(1024) void scan_top_kernel(uint32_t* __restrict__ tile_sum, uint32_t n_tiles) {
  __shared__ uint32_t sh[16];
  uint32_t carry = 0;
  for (uint32_t base = 0; base < n_tiles; base += 4096) {
    const uint32_t i = base + threadIdx.x * 4;
    uint32_t v[4], s = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) { v[k] = i + k < n_tiles ? tile_sum[i + k] : 0; s += v[k]; }
    const uint32_t incl = wave_incl_scan(s);
    if ((threadIdx.x & 63u) == 63) sh[threadIdx.x >> 6] = incl;
    __syncthreads();
    uint32_t run = carry + incl - s;
    for (uint32_t w = 0; w < 16; w++) {
      if (w < (threadIdx.x >> 6)) run += sh[w];
      carry += sh[w];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) { if (i + k < n_tiles) tile_sum[i + k] = run; run += v[k]; }
  }
}

// out[i] = sum of the items before i, *total = sum of all.  TOP: tile_sum holds the sums before each
// tile; otherwise the tiles' own sums, and a workgroup adds up those before its own.
template <class L, bool TOP>
__global__ __launch_bounds__(256) void scan_apply_kernel(L load, uint32_t n, const uint32_t* __restrict__ tile_sum,
                                                         uint32_t* __restrict__ out, uint32_t* __restrict__ total) {
  __shared__ uint32_t sh[4];
  const uint32_t first = scan_first();
  uint32_t x[kScanRows], y[kScanRows];
  scan_load(load, first, n, x, y);
  uint32_t base;
  if (TOP) {
    base = tile_sum[blockIdx.x];
  } else {
    uint32_t s = 0;
    for (uint32_t t = threadIdx.x; t < blockIdx.x; t += 256) s += tile_sum[t];
    base = block_reduce_256(s, sh);
  }
  uint32_t row[kScanRows], before[kScanRows];      // the lane's sum of a row; of the rows before it and of the lanes before it
#pragma unroll
  for (uint32_t r = 0; r < kScanRows; r++) row[r] = x[r] + y[r];
  uint32_t wave = 0;
#pragma unroll
  for (uint32_t r = 0; r < kScanRows; r += 2) {
    const uint32_t incl = wave_incl_scan(row[r] | row[r + 1] << 16), tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    before[r] = wave + (incl & 0xFFFFu) - row[r];
    wave += tot & 0xFFFFu;
    before[r + 1] = wave + (incl >> 16) - row[r + 1];
    wave += tot >> 16;
  }
  if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = wave;
  __syncthreads();
  uint32_t run = base;
  for (uint32_t w = 0; w < (threadIdx.x >> 6); w++) run += sh[w];
#pragma unroll
  for (uint32_t r = 0; r < kScanRows; r++) {
    const uint32_t i = first + r * kScanRow, at = run + before[r];
    if (i + 1 < n) *(uint2*)(out + i) = make_uint2(at, at + x[r]);
    else if (i < n) out[i] = at;
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = base + sh[0] + sh[1] + sh[2] + sh[3];
}

// One launch up to one tile, two up to kScanTop, then three: adding up the tiles before its own costs a
// workgroup up to eight reads per thread there, less than a launch between the two others.
template <class L>
static void exclusive_scan(L load, uint32_t n, uint32_t* tile_tmp, uint32_t* out, uint32_t* total, hipStream_t st) {
  const uint32_t n_tiles = n ? (n - 1) / kScanTile + 1 : 1;
  if (n_tiles > 1) hipLaunchKernelGGL(scan_tile_sums_kernel<L>, dim3(n_tiles), dim3(256), 0, st, load, n, tile_tmp);
  if (n_tiles > kScanTop) {
    hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(1024), 0, st, tile_tmp, n_tiles);
    hipLaunchKernelGGL(HIP_KERNEL_NAME(scan_apply_kernel<L, true>), dim3(n_tiles), dim3(256), 0, st, load, n, tile_tmp, out, total);
  } else {
    hipLaunchKernelGGL(HIP_KERNEL_NAME(scan_apply_kernel<L, false>), dim3(n_tiles), dim3(256), 0, st, load, n, tile_tmp, out, total);
  }
}

void scan_mask_words(const unsigned long long* mask, uint32_t n_words, uint32_t* tile_tmp, uint32_t* prefix,
                     uint32_t* total, hipStream_t st) {
  exclusive_scan(LoadPopc{mask}, n_words, tile_tmp, prefix, total, st);
}

void scan_flags(const uint8_t* flags, uint32_t n, uint32_t* tile_tmp, uint32_t* pos, uint32_t* total, hipStream_t st) {
  exclusive_scan(LoadFlag{flags}, n, tile_tmp, pos, total, st);
}

// The live boxes move to dense arrays, in index order: box b becomes box pos[b].  The old alive[]
// stays as it is: together with pos[] it translates the index a box had after the first pass
// (its rank in the mask) into the new one.
__global__ __launch_bounds__(256) void compact_boxes_kernel(uint32_t n, const uint8_t* __restrict__ alive,
                                                            const uint32_t* __restrict__ pos,
                                                            const uint32_t* __restrict__ bcell,
                                                            const uint4* __restrict__ blen, uint32_t* __restrict__ cell2,
                                                            uint4* __restrict__ len2, uint8_t* __restrict__ alive2) {
  const uint32_t b = blockIdx.x * 256u + threadIdx.x;
  if (b >= n || !alive[b]) return;
  const uint32_t j = pos[b];
  cell2[j] = bcell[b];
  len2[j] = blen[b];
  alive2[j] = kLive;
}

void launch_compact_boxes(uint32_t n, const uint8_t* alive, const uint32_t* pos, const uint32_t* bcell, const void* blen,
                          uint32_t* cell2, void* len2, uint8_t* alive2, hipStream_t st) {
  hipLaunchKernelGGL(compact_boxes_kernel, dim3((n + 255) / 256), dim3(256), 0, st, n, alive, pos, bcell, (const uint4*)blen,
                     cell2, (uint4*)len2, alive2);
}

// ---------------------------------------------------------------- boxes of pass 0

// A wave of the word-by-word kernels takes this many consecutive mask words: 64 (one per lane)
// on large tables, few on small ones, which would otherwise occupy a handful of waves for long.
static uint32_t words_per_wave(uint32_t n_words) { return n_words >= (1u << 21) ? 64u : 8u; }

// General form (any stride): a flagged cell opens the box whose index is its rank in the table-order
// mask (prefix sums), and the box runs to the next flagged cell of the line or to the line's end.
// A wave takes wpw consecutive words (a word and its prefix sum per lane) and their boxes 64 at a
// time, a lane each: the word by a search in the prefix sums, the cell as its n-th flag.  The lanes
// write consecutive boxes.  (A lane per cell, most of which open no box, with the words read one
// after the other, took 145 us for 2.4 M boxes in 41 M cells, this 26; 51 MB of boxes and 8 MB of words
// take 11.  8 words a wave on small tables, where 64 would leave the chip idle.)
__global__ __launch_bounds__(256) void make_boxes_kernel(Geo g, uint32_t a0, uint32_t n_words, uint32_t wpw,
                                                         const unsigned long long* __restrict__ mask,
                                                         const uint32_t* __restrict__ prefix,
                                                         uint32_t* __restrict__ bcell, uint4* __restrict__ blen,
                                                         uint8_t* __restrict__ alive) {
  __shared__ unsigned long long s_mask[256];
  __shared__ uint32_t s_first[256];
  const uint32_t lane = threadIdx.x & 63u, at = threadIdx.x & ~63u;
  const uint32_t w0 = (blockIdx.x * 4u + (threadIdx.x >> 6)) * wpw;
  const bool mine = lane < wpw && w0 + lane < n_words;
  const unsigned long long mv = mine ? mask[w0 + lane] : 0ull;
  const uint32_t pv = mine ? prefix[w0 + lane] : 0xFFFFFFFFu;
  const uint32_t id0 = (uint32_t)__shfl((int)pv, 0);
  s_mask[threadIdx.x] = mv;
  s_first[threadIdx.x] = pv - id0;
  __syncthreads();
  if (w0 >= n_words) return;
  const uint32_t last = min(wpw, n_words - w0) - 1u;
  const uint32_t n_boxes = s_first[at + last] + (uint32_t)__popcll(s_mask[at + last]);
  const uint32_t s0 = g.stride[a0], e0 = g.ext[a0];
  // a power-of-two stride: the line's cells sit at the same bit positions (mod s0) of every word
  const bool in_words = (s0 & (s0 - 1u)) == 0 && s0 <= 32u;
  const unsigned long long P = s0 == 1 ? ~0ull : s0 == 2 ? 0x5555555555555555ull : s0 == 4 ? 0x1111111111111111ull
                             : s0 == 8 ? 0x0101010101010101ull : s0 == 16 ? 0x0001000100010001ull : 0x0000000100000001ull;
  const uint32_t shift = (a0 & 3u) * 8u;
  for (uint32_t i = lane; i < n_boxes; i += 64u) {
    uint32_t t = 0;                                       // the last word whose boxes start at or before box i (words without any come before it)
#pragma unroll
    for (uint32_t d = 32; d > 0; d >>= 1)
      if (t + d <= last && s_first[at + t + d] <= i) t += d;
    const unsigned long long tm = s_mask[at + t];
    const uint32_t bit0 = nth_bit(tm, i - s_first[at + t]);
    const uint32_t word = w0 + t, cell = word * 64u + bit0;
    const uint32_t j = (cell / s0) % e0;
    const uint32_t R = e0 - 1u - j;                       // cells after this one on the line
    uint32_t len = R + 1u;
    if (in_words) {
      // the next flagged one is a mask, a count of trailing zeros and a division away
      const unsigned long long same = P << (bit0 % s0);
      unsigned long long m = tm & same & ~((2ull << bit0) - 1ull);      // this word: only the cells after this one
      for (uint32_t k = word;; m = (k - w0 <= last ? s_mask[at + k - w0] : mask[k]) & same) {
        if (m) {
          const uint32_t run = (k * 64u + (uint32_t)__builtin_ctzll(m) - cell) / s0;
          if (run <= R) len = run;
          break;
        }
        if ((k * 64u + 63u - cell) / s0 >= R) break;      // the line ends inside this word
        k++;
      }
    } else {
      for (len = 1; len <= R; len++) {
        const uint32_t c2 = cell + len * s0;
        if ((mask[c2 >> 6] >> (c2 & 63u)) & 1ull) break;
      }
    }
    uint32_t L[4] = {0x01010101u, 0x01010101u, 0x01010101u, 0x01010101u};
    const uint32_t w = (0x01010101u & ~(0xFFu << shift)) | (len << shift);
    L[0] = (a0 >> 2) == 0 ? w : L[0];
    L[1] = (a0 >> 2) == 1 ? w : L[1];
    L[2] = (a0 >> 2) == 2 ? w : L[2];
    L[3] = (a0 >> 2) == 3 ? w : L[3];
    bcell[id0 + i] = cell;
    blen[id0 + i] = make_uint4(L[0], L[1], L[2], L[3]);
    alive[id0 + i] = kLive;
  }
}

// The same for lines whose stride is a multiple of 64 cells, word by word of the table-order
// mask: a wave takes 64 consecutive words (lane t fetches word t and its prefix sum) and then,
// for every word that flags a cell, stands with its 64 lanes on the word's 64 cells.  These lie
// on 64 consecutive lines at the same step, so the lanes read consecutive words of the line-major
// mask (for the run's end), and the boxes they open have consecutive indices: all of a wave's
// reads and writes are contiguous stretches.
constexpr int kBoxWords = 4;

__global__ __launch_bounds__(256) void make_boxes_wave_kernel(Geo g, uint32_t a0, uint32_t n_words, uint32_t wpw,
                                                              const unsigned long long* __restrict__ mask,
                                                              const uint32_t* __restrict__ prefix,
                                                              const unsigned long long* __restrict__ line,
                                                              const unsigned long long* __restrict__ col, uint32_t a1,
                                                              uint32_t* __restrict__ bcell, uint4* __restrict__ blen,
                                                              uint8_t* __restrict__ alive) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t w0 = (blockIdx.x * 4u + (threadIdx.x >> 6)) * wpw;
  if (w0 >= n_words) return;
  const uint32_t s0 = g.stride[a0], e0 = g.ext[a0], n_lines = g.n / e0, se = s0 * e0;
  const uint32_t shift = (a0 & 3u) * 8u;
  const bool mine = lane < wpw && w0 + lane < n_words;
  const unsigned long long mv = mine ? mask[w0 + lane] : 0ull;
  const uint32_t pv = mine ? prefix[w0 + lane] : 0u;
  // kBoxWords words at a time, so that their reads of the line-major mask are in flight together
  unsigned long long todo = __ballot(mv != 0);
  while (todo) {
    uint32_t id[kBoxWords], cell[kBoxWords], j[kBoxWords], q[kBoxWords], c1[kBoxWords];
    bool head[kBoxWords];
    unsigned long long lm[kBoxWords], cw[kBoxWords];
#pragma unroll
    for (int u = 0; u < kBoxWords; u++) {
      const bool any = todo != 0;
      const uint32_t t = any ? (uint32_t)__ffsll((long long)todo) - 1u : 0u;
      todo &= todo - 1;                 // 0 stays 0
      const unsigned long long m = any ? readlane64(mv, t) : 0ull;
      const uint32_t pf = (uint32_t)__builtin_amdgcn_readlane((int)pv, (int)t);
      const uint32_t cell0 = (w0 + t) * 64u;               // the word's first cell; all 64 share the step j
      const uint32_t hi = cell0 / se, rem = cell0 - hi * se;
      j[u] = rem / s0;
      q[u] = hi * s0 + (rem - j[u] * s0) + lane;
      cell[u] = cell0 + lane;
      id[u] = pf + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
      head[u] = (m >> lane) & 1ull;
      lm[u] = head[u] ? line[(size_t)(j[u] >> 6) * n_lines + q[u]] : 0ull;
      cw[u] = 0; c1[u] = 0;
      if (col) {                        // the runs behind this box on a1 that were folded into it
        const uint32_t s1 = g.stride[a1], e1 = g.ext[a1], se1 = s1 * e1;
        const uint32_t hi1 = cell0 / se1, rem1 = cell0 - hi1 * se1;
        c1[u] = rem1 / s1;
        cw[u] = head[u] ? col[(size_t)hi1 * s1 + (rem1 - c1[u] * s1) + lane] : 0ull;
      }
    }
#pragma unroll
    for (int u = 0; u < kBoxWords; u++) {
      if (head[u]) {
        uint32_t end = e0;                                 // the run ends at the line's next flagged cell
        unsigned long long w = lm[u] & ~((2ull << (j[u] & 63u)) - 1ull);
        for (uint32_t k = j[u] >> 6;;) {
          if (w) { end = k * 64u + (uint32_t)__ffsll((long long)w) - 1u; break; }
          if (++k * 64u >= e0) break;
          w = line[(size_t)k * n_lines + q[u]];
        }
        uint32_t L[4] = {0x01010101u, 0x01010101u, 0x01010101u, 0x01010101u};
        const uint32_t lw = (0x01010101u & ~(0xFFu << shift)) | ((end - j[u]) << shift);
        L[0] = (a0 >> 2) == 0 ? lw : L[0];
        L[1] = (a0 >> 2) == 1 ? lw : L[1];
        L[2] = (a0 >> 2) == 2 ? lw : L[2];
        L[3] = (a0 >> 2) == 3 ? lw : L[3];
        if (col) {
          // bit c of the column word: the run at step c was folded into the one before it
          const unsigned long long above = c1[u] >= 63u ? 0ull : cw[u] >> (c1[u] + 1u);
          const uint32_t more = (uint32_t)__ffsll((long long)~above) - 1u;
          const uint32_t add = more << ((a1 & 3u) * 8u);                       // the byte holds 1
          L[0] += (a1 >> 2) == 0 ? add : 0u;
          L[1] += (a1 >> 2) == 1 ? add : 0u;
          L[2] += (a1 >> 2) == 2 ? add : 0u;
          L[3] += (a1 >> 2) == 3 ? add : 0u;
        }
        bcell[id[u]] = cell[u];
        blen[id[u]] = make_uint4(L[0], L[1], L[2], L[3]);
        alive[id[u]] = kLive;
      }
    }
  }
}

// ---------------------------------------------------------------- the second merge axis, on cells
// The first generic pass would link every run of pass 0 to the run one step further on the second
// merge axis a1 when both have the same value and the same extent on a0 (they differ in no other
// extent yet).  For an a1 that lies outside a0, with a stride of whole mask words and at most 64
// steps, this is decided on the cells before any box exists: a run head whose predecessor on a1
// heads an equal run loses its flag and sets the bit of its step in the word of its column (the
// cells that differ only on a1), from which make_boxes reads the length of the chain.  runs = the
// mask of pass 0, mask2 = the heads of boxes, col = one word per column, zero before.
constexpr int kSecondWords = 4;

// first = the line's mask word that holds step j
__device__ __forceinline__ uint32_t run_end(unsigned long long first, const unsigned long long* __restrict__ line,
                                            uint32_t n_lines, uint32_t e0, uint32_t j, uint32_t q) {
  unsigned long long w = first & ~((2ull << (j & 63u)) - 1ull);
  for (uint32_t k = j >> 6;;) {
    if (w) return k * 64u + (uint32_t)__ffsll((long long)w) - 1u;
    if (++k * 64u >= e0) return e0;
    w = line[(size_t)k * n_lines + q];
  }
}

template <bool COST>
__global__ __launch_bounds__(256) void second_axis_kernel(Geo g, uint32_t a0, uint32_t a1, uint32_t n_words, uint32_t wpw,
                                                          const unsigned long long* __restrict__ runs,
                                                          const unsigned long long* __restrict__ line,
                                                          const unsigned long long* __restrict__ fitmap,
                                                          const uint64_t* __restrict__ cost, const uint16_t* __restrict__ arg,
                                                          const uint32_t* __restrict__ axis_sizes,
                                                          unsigned long long* __restrict__ mask2,
                                                          unsigned long long* __restrict__ col) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t w0 = (blockIdx.x * 4u + (threadIdx.x >> 6)) * wpw;
  if (w0 >= n_words) return;
  const uint32_t s0 = g.stride[a0], e0 = g.ext[a0], n_lines = g.n / e0, se = s0 * e0;
  const uint32_t s1 = g.stride[a1], e1 = g.ext[a1], d = s1 >> 6, back = s1 / se * s0, se1 = s1 * e1;
  const bool mine = lane < wpw && w0 + lane < n_words;
  const unsigned long long mv = mine ? runs[w0 + lane] : 0ull;
  unsigned long long out = mv;
  // kSecondWords words at a time, each stage's reads side by side
  unsigned long long todo = __ballot(mv != 0);
  while (todo) {
    uint32_t t[kSecondWords], w[kSecondWords], c1[kSecondWords];
    unsigned long long m[kSecondWords], cand[kSecondWords], fc[kSecondWords], fp[kSecondWords];
#pragma unroll
    for (int u = 0; u < kSecondWords; u++) {
      const bool any = todo != 0;
      t[u] = any ? (uint32_t)__ffsll((long long)todo) - 1u : 0u;
      todo &= todo - 1;                 // 0 stays 0
      m[u] = any ? readlane64(mv, t[u]) : 0ull;
      w[u] = w0 + t[u];
      c1[u] = (w[u] * 64u / s1) % e1;   // the word's 64 cells share it
      const bool has = m[u] != 0 && c1[u] > 0;
      cand[u] = has ? m[u] & runs[w[u] - d] : 0ull;       // the cell before on a1 heads a run as well
      fc[u] = has ? fitmap[w[u]] : 0ull;
      fp[u] = has ? fitmap[w[u] - d] : 0ull;
    }
    bool me[kSecondWords];
    uint64_t vc[kSecondWords], vp[kSecondWords];
#pragma unroll
    for (int u = 0; u < kSecondWords; u++) {
      me[u] = (cand[u] >> lane) & 1ull;
      const uint32_t cell = w[u] * 64u + lane;
      const bool rc = me[u] && ((fc[u] >> lane) & 1ull), rp = me[u] && ((fp[u] >> lane) & 1ull);
      if (COST) {
        vc[u] = rc ? cost[cell] : kInf;
        vp[u] = rp ? cost[cell - s1] : kInf;
      } else {
        vc[u] = rc ? (uint64_t)arg[cell] : (uint64_t)kNone;
        vp[u] = rp ? (uint64_t)arg[cell - s1] : (uint64_t)kNone;
      }
    }
    bool same[kSecondWords];
    uint32_t j[kSecondWords], q[kSecondWords];
    unsigned long long lc[kSecondWords], lp[kSecondWords];
#pragma unroll
    for (int u = 0; u < kSecondWords; u++) {
      if (COST) {
        const uint32_t z1 = (axis_sizes && c1[u]) ? axis_sizes[c1[u] - 1] : 1u, z2 = axis_sizes ? axis_sizes[c1[u]] : 1u;
        same[u] = me[u] && norm_equal(vp[u], z1, vc[u], z2);
      } else {
        same[u] = me[u] && vp[u] == vc[u];
      }
      const uint32_t cell0 = w[u] * 64u, hi = cell0 / se, rem = cell0 - hi * se;
      j[u] = rem / s0;
      q[u] = hi * s0 + (rem - j[u] * s0) + lane;
      const size_t at = (size_t)(j[u] >> 6) * n_lines + q[u];
      lc[u] = same[u] ? line[at] : 0ull;
      lp[u] = same[u] ? line[at - back] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < kSecondWords; u++) {
      if (same[u])        // equal extents on a0: both runs end at the same step
        same[u] = run_end(lc[u], line, n_lines, e0, j[u], q[u]) == run_end(lp[u], line, n_lines, e0, j[u], q[u] - back);
      if (same[u]) {
        const uint32_t cell0 = w[u] * 64u, hi1 = cell0 / se1, rem1 = cell0 - hi1 * se1;
        atomicOr(&col[(size_t)hi1 * s1 + (rem1 - c1[u] * s1) + lane], 1ull << c1[u]);
      }
      const unsigned long long gone = __ballot(same[u]);
      if (m[u] && lane == t[u]) out = m[u] & ~gone;
    }
  }
  if (mine) mask2[w0 + lane] = out;
}

// ---------------------------------------------------------------- pass on axis a
__device__ __forceinline__ uint32_t len_byte(const uint4& L, uint32_t a) {
  const uint32_t w = a < 4 ? L.x : a < 8 ? L.y : a < 12 ? L.z : L.w;
  return (w >> ((a & 3u) * 8)) & 0xFFu;
}

// Every box still has extent 1 on axis a when its pass comes (an axis is merged once).  Most
// boxes differ in value from the cell past their end, so the values are compared first and the
// extents are read only for the few that pass.  block_linked[workgroup] tells the absorb step
// whether any of the workgroup's boxes got a successor.  After the compaction the mask still
// ranks boxes by their old index: old_alive / remap translate it (nullptr before).
template <bool COST>
__global__ __launch_bounds__(256) void link_kernel(Geo g, uint32_t a, uint8_t stamp, uint32_t n_boxes,
                                                   const uint8_t* __restrict__ old_alive,
                                                   const uint32_t* __restrict__ remap,
                                                   const uint32_t* __restrict__ bcell, const uint4* __restrict__ blen,
                                                   uint8_t* alive,
                                                   uint32_t* __restrict__ next, uint32_t* __restrict__ block_linked,
                                                   const unsigned long long* __restrict__ mask,
                                                   const uint32_t* __restrict__ prefix,
                                                   const uint64_t* __restrict__ cost, const uint16_t* __restrict__ arg,
                                                   const uint32_t* __restrict__ axis_sizes) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  const uint32_t b = i < n_boxes ? i : 0u;
  const bool live = i < n_boxes && alive[b];
  uint32_t nxt = 0xFFFFFFFFu;
  if (live) {
    const uint32_t cell = bcell[b];
    const uint32_t sa = g.stride[a], ea = g.ext[a];
    const uint32_t ca = (cell / sa) % ea;
    if (ca + 1 < ea) {
      const uint32_t s = cell + sa;
      bool same;
      if (COST) {
        const uint32_t s1 = axis_sizes ? axis_sizes[ca] : 1u, s2 = axis_sizes ? axis_sizes[ca + 1] : 1u;
        same = norm_equal(cost[cell], s1, cost[s], s2);
      } else {
        same = arg[cell] == arg[s];
      }
      if (same) {
        const unsigned long long m = mask[s >> 6];
        if ((m >> (s & 63u)) & 1ull) {
          uint32_t o = prefix[s >> 6] + (uint32_t)__popcll(m & ((1ull << (s & 63u)) - 1ull));
          bool there = true;
          if (remap) { there = old_alive[o]; o = there ? remap[o] : 0u; }
          if (there && alive[o]) {
            const uint4 L = blen[b], M = blen[o];     // equal on a as well: both 1
            if (L.x == M.x && L.y == M.y && L.z == M.z && L.w == M.w) {
              nxt = o;
              alive[o] = kLive | stamp;
            }
          }
        }
      }
    }
    next[b] = nxt;
  }
  const int any = __syncthreads_or(nxt != 0xFFFFFFFFu);
  if (threadIdx.x == 0) block_linked[blockIdx.x] = (uint32_t)any;
}

__global__ __launch_bounds__(256) void absorb_kernel(uint32_t a, uint8_t stamp, uint32_t n_boxes,
                                                     uint8_t* __restrict__ blen_bytes,
                                                     uint8_t* alive,
                                                     const uint32_t* __restrict__ next,
                                                     const uint32_t* __restrict__ block_linked) {
  if (!block_linked[blockIdx.x]) return;       // no box of this workgroup got a successor: no chain starts here
  const uint32_t b = blockIdx.x * 256u + threadIdx.x;
  if (b >= n_boxes) return;
  uint32_t s = next[b];
  if (s == 0xFFFFFFFFu || !alive[b] || alive[b] == (kLive | stamp)) return;   // only heads of chains of two or more
  uint32_t tot = blen_bytes[(size_t)b * 16 + a];
  for (; s != 0xFFFFFFFFu; s = next[s]) {
    tot += blen_bytes[(size_t)s * 16 + a];
    alive[s] = 0;
  }
  blen_bytes[(size_t)b * 16 + a] = (uint8_t)tot;
}

void launch_head_flags(const Geo& g, uint32_t a0, const uint64_t* cost, const uint16_t* arg, const uint32_t* fitmap,
                       const uint32_t* axis_sizes,
                       unsigned long long* maskD, unsigned long long* maskC, unsigned long long* lineD,
                       unsigned long long* lineC, hipStream_t st) {
  const uint32_t n_lines = g.n / g.ext[a0];
  const uint32_t blocks = (n_lines + 255) / 256;
  if (g.stride[a0] % 64 == 0)
    hipLaunchKernelGGL(head_flags_wave_kernel, dim3((blocks + 4 * kHeadSpread - 1) / (4 * kHeadSpread) * (4 * kHeadSpread)), dim3(256), 0, st, g, a0, cost, arg,
                       (const unsigned long long*)fitmap, axis_sizes, maskD, maskC, lineD, lineC);
  else
    hipLaunchKernelGGL(head_flags_kernel, dim3((g.n + 256 * kCellWords - 1) / (256 * kCellWords)), dim3(256), 0, st, g, a0, cost, arg,
                       (const unsigned long long*)fitmap, axis_sizes, maskD, maskC);
}

void launch_second_axis(const Geo& g, uint32_t a0, uint32_t a1, bool is_cost, const unsigned long long* runs,
                        const unsigned long long* line, const uint32_t* fitmap, const uint64_t* cost, const uint16_t* arg,
                        const uint32_t* axis_sizes, unsigned long long* mask2, unsigned long long* col, hipStream_t st) {
  const uint32_t n_words = g.n / 64;
  const uint32_t wpw = words_per_wave(n_words);
  const dim3 grid((n_words + 4 * wpw - 1) / (4 * wpw));
  if (is_cost)
    hipLaunchKernelGGL(second_axis_kernel<true>, grid, dim3(256), 0, st, g, a0, a1, n_words, wpw, runs, line,
                       (const unsigned long long*)fitmap, cost, arg, axis_sizes, mask2, col);
  else
    hipLaunchKernelGGL(second_axis_kernel<false>, grid, dim3(256), 0, st, g, a0, a1, n_words, wpw, runs, line,
                       (const unsigned long long*)fitmap, cost, arg, axis_sizes, mask2, col);
}

void launch_make_boxes(const Geo& g, uint32_t a0, const unsigned long long* mask, const uint32_t* prefix,
                       const unsigned long long* line, const unsigned long long* col, uint32_t a1, uint32_t* bcell,
                       void* blen, uint8_t* alive, hipStream_t st) {
  const uint32_t n_words = (g.n + 63) / 64;
  if (g.stride[a0] % 64 == 0) {
    const uint32_t wpw = words_per_wave(n_words);
    hipLaunchKernelGGL(make_boxes_wave_kernel, dim3((n_words + 4 * wpw - 1) / (4 * wpw)), dim3(256), 0, st, g, a0, n_words, wpw, mask, prefix,
                       line, col, a1, bcell, (uint4*)blen, alive);
  } else {
    const uint32_t wpw = n_words >= (1u << 18) ? 64u : 8u;        // 4,096 waves from there on
    hipLaunchKernelGGL(make_boxes_kernel, dim3((n_words + 4 * wpw - 1) / (4 * wpw)), dim3(256), 0, st, g, a0, n_words, wpw, mask, prefix,
                       bcell, (uint4*)blen, alive);
  }
}

void launch_axis_pass(const Geo& g, uint32_t a, uint8_t stamp, bool is_cost, uint32_t n_boxes, const uint8_t* old_alive,
                      const uint32_t* remap, const uint32_t* bcell, void* blen, uint8_t* alive, uint32_t* next,
                      uint32_t* block_linked, const unsigned long long* mask, const uint32_t* prefix, const uint64_t* cost,
                      const uint16_t* arg, const uint32_t* axis_sizes, hipStream_t st) {
  const uint32_t blocks = (n_boxes + 255) / 256;
  if (is_cost)
    hipLaunchKernelGGL(link_kernel<true>, dim3(blocks), dim3(256), 0, st, g, a, stamp, n_boxes, old_alive, remap, bcell,
                       (const uint4*)blen, alive, next, block_linked, mask, prefix, cost, arg, axis_sizes);
  else
    hipLaunchKernelGGL(link_kernel<false>, dim3(blocks), dim3(256), 0, st, g, a, stamp, n_boxes, old_alive, remap, bcell,
                       (const uint4*)blen, alive, next, block_linked, mask, prefix, cost, arg, axis_sizes);
  hipLaunchKernelGGL(absorb_kernel, dim3(blocks), dim3(256), 0, st, a, stamp, n_boxes, (uint8_t*)blen, alive, next,
                     block_linked);
}

// ---------------------------------------------------------------- the last passes, in one
// The merge order ends with the axes of the layout and dtype bits, which are also the innermost
// coordinates: extent 2 and a stride of at most 32 cells, so a box and the one it could merge
// with on such an axis have their low corners in the same 64-cell word of the mask, and no chain
// is longer than two.  A wave stands with its lanes on the cells of a word, holds the live boxes
// that start there in registers, and runs all those passes with lane exchanges: one read and at
// most one write of every box instead of one per pass.
constexpr int kTailWords = 4;

template <bool COST>
__global__ __launch_bounds__(256) void tail_pairs_kernel(TailAxes T, uint32_t n_words, uint32_t wpw,
                                                         const unsigned long long* __restrict__ mask,
                                                         const uint32_t* __restrict__ prefix,
                                                         const uint8_t* __restrict__ old_alive,
                                                         const uint32_t* __restrict__ remap, uint4* __restrict__ blen,
                                                         uint8_t* __restrict__ alive, const uint64_t* __restrict__ cost,
                                                         const uint16_t* __restrict__ arg) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t w0 = (blockIdx.x * 4u + (threadIdx.x >> 6)) * wpw;
  if (w0 >= n_words) return;
  const bool mine = lane < wpw && w0 + lane < n_words;
  const unsigned long long mv = mine ? mask[w0 + lane] : 0ull;
  const uint32_t pv = mine ? prefix[w0 + lane] : 0u;
  // kTailWords words at a time, their reads side by side: every read is a trip to memory, and a
  // word needs four of them in a row (old alive, new index, live, extents and value)
  unsigned long long todo = __ballot(mv != 0);
  while (todo) {
    uint32_t id[kTailWords], cell[kTailWords];
    bool live[kTailWords];
#pragma unroll
    for (int u = 0; u < kTailWords; u++) {
      const bool any = todo != 0;
      const uint32_t t = any ? (uint32_t)__ffsll((long long)todo) - 1u : 0u;
      todo &= todo - 1;                 // 0 stays 0
      const unsigned long long m = any ? readlane64(mv, t) : 0ull;
      const uint32_t pf = (uint32_t)__builtin_amdgcn_readlane((int)pv, (int)t);
      cell[u] = (w0 + t) * 64u + lane;
      id[u] = pf + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
      live[u] = (m >> lane) & 1ull;
    }
    if (remap) {                       // the mask ranks boxes by the index they had before the compaction
#pragma unroll
      for (int u = 0; u < kTailWords; u++) live[u] = live[u] && old_alive[id[u]];
#pragma unroll
      for (int u = 0; u < kTailWords; u++) id[u] = live[u] ? remap[id[u]] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kTailWords; u++) live[u] = live[u] && alive[id[u]];
    uint4 L[kTailWords];
    uint64_t v[kTailWords];
#pragma unroll
    for (int u = 0; u < kTailWords; u++) {
      L[u] = live[u] ? blen[id[u]] : make_uint4(0, 0, 0, 0);
      // the two boxes of a pair start in the same shape, so equal normalised costs = equal costs
      v[u] = 0;
      if (live[u]) v[u] = COST ? cost[cell[u]] : (uint64_t)arg[cell[u]];
    }
#pragma unroll
    for (int u = 0; u < kTailWords; u++) {
      if (!__any(live[u])) continue;
      bool changed = false, died = false;
      for (uint32_t k = 0; k < T.n; k++) {
        const uint32_t st = T.stride[k], a = T.axis[k];
        const int p_live = __shfl_down((int)live[u], st, 64);
        const uint32_t p_lo = __shfl_down((uint32_t)v[u], st, 64), p_hi = __shfl_down((uint32_t)(v[u] >> 32), st, 64);
        const uint32_t px = __shfl_down(L[u].x, st, 64), py = __shfl_down(L[u].y, st, 64);
        const uint32_t pz = __shfl_down(L[u].z, st, 64), pw = __shfl_down(L[u].w, st, 64);
        const bool low = (lane & st) == 0;             // coordinate 0 on this axis: lane + st is in the same word
        const bool merge = low && live[u] && p_live && (uint32_t)v[u] == p_lo && (uint32_t)(v[u] >> 32) == p_hi &&
                           L[u].x == px && L[u].y == py && L[u].z == pz && L[u].w == pw;
        if (merge) {
          const uint32_t one = 1u << ((a & 3u) * 8u);
          L[u].x += (a >> 2) == 0 ? one : 0u;
          L[u].y += (a >> 2) == 1 ? one : 0u;
          L[u].z += (a >> 2) == 2 ? one : 0u;
          L[u].w += (a >> 2) == 3 ? one : 0u;
          changed = true;
        }
        const int absorbed = __shfl_up((int)merge, st, 64);
        if (!low && absorbed) { live[u] = false; died = true; }
      }
      if (changed) blen[id[u]] = L[u];
      if (died) alive[id[u]] = 0;
    }
  }
}

void launch_tail_pairs(const TailAxes& T, bool is_cost, uint32_t n_words, const unsigned long long* mask,
                       const uint32_t* prefix, const uint8_t* old_alive, const uint32_t* remap, void* blen, uint8_t* alive,
                       const uint64_t* cost, const uint16_t* arg, hipStream_t st) {
  const uint32_t wpw = words_per_wave(n_words), blocks = (n_words + 4 * wpw - 1) / (4 * wpw);
  if (is_cost)
    hipLaunchKernelGGL(tail_pairs_kernel<true>, dim3(blocks), dim3(256), 0, st, T, n_words, wpw, mask, prefix, old_alive, remap,
                       (uint4*)blen, alive, cost, arg);
  else
    hipLaunchKernelGGL(tail_pairs_kernel<false>, dim3(blocks), dim3(256), 0, st, T, n_words, wpw, mask, prefix, old_alive, remap,
                       (uint4*)blen, alive, cost, arg);
}

// ---------------------------------------------------------------- final lists
// Binary gcd (shifts and subtractions: a 64-bit remainder is a long software routine here).
__device__ __forceinline__ uint64_t gcd_u64(uint64_t a, uint64_t b) {
  if (a == 0) return b;
  if (b == 0) return a;
  const int shift = __builtin_ctzll(a | b);
  a >>= __builtin_ctzll(a);
  do {
    b >>= __builtin_ctzll(b);
    if (a > b) { const uint64_t t = a; a = b; b = t; }
    b -= a;
  } while (b);
  return a << shift;
}

template <bool COST>
__global__ __launch_bounds__(256) void emit_kernel(Geo g, const DevParams* __restrict__ P,
                                                   uint32_t n_boxes,
                                                   const uint32_t* __restrict__ bcell, const uint4* __restrict__ blen,
                                                   const uint8_t* __restrict__ alive, const uint32_t* __restrict__ pos,
                                                   const uint64_t* __restrict__ cost, const uint16_t* __restrict__ arg,
                                                   uint32_t* __restrict__ fcell, uint4* __restrict__ flen,
                                                   uint64_t* __restrict__ fv0, uint64_t* __restrict__ fv1) {
  const uint32_t b = blockIdx.x * 256u + threadIdx.x;
  if (b >= n_boxes || !alive[b]) return;
  const uint32_t o = pos[b], cell = bcell[b];
  fcell[o] = cell;
  flen[o] = blen[b];
  if (COST) {
    const uint64_t c = cost[cell];
    if (c == kInf) { fv0[o] = kInf; fv1[o] = 0; }
    else {
      uint64_t vol = 1;
#pragma unroll
      for (int d = 0; d < 4; d++) vol *= P->sizes[d][(cell / g.stride[d]) % g.ext[d]];
      const uint64_t q = gcd_u64(c, vol);
      fv0[o] = c / q; fv1[o] = vol / q;
    }
  } else {
    fv0[o] = arg[cell]; fv1[o] = 0;
  }
}

void launch_emit(const Geo& g, const DevParams* P, bool is_cost, uint32_t n_boxes, const uint32_t* bcell,
                 const void* blen,
                 const uint8_t* alive, const uint32_t* pos, const uint64_t* cost, const uint16_t* arg, uint32_t* fcell,
                 void* flen, uint64_t* fv0, uint64_t* fv1, hipStream_t st) {
  const uint32_t blocks = (n_boxes + 255) / 256;
  if (is_cost)
    hipLaunchKernelGGL(emit_kernel<true>, dim3(blocks), dim3(256), 0, st, g, P, n_boxes, bcell, (const uint4*)blen,
                       alive, pos, cost, arg, fcell, (uint4*)flen, fv0, fv1);
  else
    hipLaunchKernelGGL(emit_kernel<false>, dim3(blocks), dim3(256), 0, st, g, P, n_boxes, bcell, (const uint4*)blen,
                       alive, pos, cost, arg, fcell, (uint4*)flen, fv0, fv1);
}

// The records of a final list, as the caller gets them: 80 bytes each (lo[16], hi[16] of 16 bits, then
// v0, v1), 16 bytes per lane, so that a wave writes one contiguous stretch.  out: pinned host memory.
// Bound by the link and by the host's copy out of the pinned block.  The lists of a pipeline's three
// tables (15.7 M Specs, solved and taken to the host): 7.2 ms in all; 16.6 ms when the host expanded
// them out of four copies into pageable memory.
__global__ __launch_bounds__(256) void expand_boxes_kernel(Geo g, uint32_t n, const uint32_t* __restrict__ fcell, const uint4* __restrict__ flen,
                                                           const uint64_t* __restrict__ fv0, const uint64_t* __restrict__ fv1,
                                                           uint4* __restrict__ out) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  const uint32_t b = i / 5u, piece = i - b * 5u;
  if (b >= n) return;
  if (piece == 4) {
    const uint64_t v0 = fv0[b], v1 = fv1[b];
    out[i] = make_uint4((uint32_t)v0, (uint32_t)(v0 >> 32), (uint32_t)v1, (uint32_t)(v1 >> 32));
    return;
  }
  const uint32_t cell = fcell[b], half = piece & 1u;         // axes 0..7 or 8..15
  const bool hi = piece >= 2;
  const uint4 L = flen[b];
  const uint32_t l0 = half ? L.z : L.x, l1 = half ? L.w : L.y;
  uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
  for (uint32_t k = 0; k < 8; k++) {
    const uint32_t a = half * 8u + k;
    if (a >= g.ndim) break;
    const uint32_t stride = half ? g.stride[8 + k] : g.stride[k], ext = half ? g.ext[8 + k] : g.ext[k];
    uint32_t x = (cell / stride) % ext;
    if (hi) x += (((k < 4 ? l0 : l1) >> (8u * (k & 3u))) & 0xFFu) - 1u;
    w[k >> 1] |= (x & 0xFFFFu) << (16u * (k & 1u));
  }
  out[i] = make_uint4(w[0], w[1], w[2], w[3]);
}

hipError_t launch_expand_boxes(const Geo& g, uint32_t n, const uint32_t* fcell, const void* flen, const uint64_t* fv0, const uint64_t* fv1, void* out,
                         hipStream_t st) {
  if (!n) return hipSuccess;
  return launch_checked(expand_boxes_kernel, dim3((n * 5u + 255u) / 256u), dim3(256), st, g, n, fcell, (const uint4*)flen, fv0, fv1, (uint4*)out);
}

// ---------------------------------------------------------------- query
__global__ __launch_bounds__(256) void gather_kernel(const uint64_t* __restrict__ idx, uint32_t n,
                                                     const uint64_t* __restrict__ cost, const uint16_t* __restrict__ arg,
                                                     uint64_t* __restrict__ cost_out, uint16_t* __restrict__ arg_out) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  cost_out[i] = cost[idx[i]];
  arg_out[i] = arg[idx[i]];
}

hipError_t launch_gather(const uint64_t* idx, uint32_t n, const uint64_t* cost, const uint16_t* arg, uint64_t* cost_out,
                   uint16_t* arg_out, hipStream_t st) {
  return launch_checked(gather_kernel, dim3((n + 255) / 256), dim3(256), st, idx, n, cost, arg, cost_out, arg_out);
}

// One lane follows a program through one table: entry, rewrite, the Spec it leads to, as long as that
// Spec lies in this table and differs only in what the rewrite id names (a Move to another level,
// perhaps in another layout or type; a tile loop).  Bound by the latency of two reads a step, a few
// microseconds; with a launch, copies and the host's wait around every step, and the whole walk once
// more to count its nodes, a program of 18 rewrites took 1.35 ms, now 0.06.
__global__ __launch_bounds__(64) void chain_kernel(ChainWalk w, const uint64_t* __restrict__ cost, const uint16_t* __restrict__ arg,
                                                   ChainEntry* __restrict__ out, uint32_t* __restrict__ n_out) {
  __shared__ uint32_t x[16], ext[16], stride[16];
  __shared__ int lay_axis[5], dt_axis[5];
  if (threadIdx.x < 16) {
    x[threadIdx.x] = w.x[threadIdx.x];
    ext[threadIdx.x] = w.g.ext[threadIdx.x];
    stride[threadIdx.x] = w.g.stride[threadIdx.x];
  }
  if (threadIdx.x < 5) {
    lay_axis[threadIdx.x] = w.lay_axis[threadIdx.x];
    dt_axis[threadIdx.x] = w.dt_axis[threadIdx.x];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  uint32_t cell = w.cell, n = 0;
  // axis a's coordinate becomes v; false if there is no such cell
  auto go = [&](uint32_t a, uint32_t v) -> bool {
    if (a >= w.g.ndim || v >= ext[a]) return false;
    cell += (v - x[a]) * stride[a];
    x[a] = v;
    return true;
  };
  while (n < kChainMost) {
    const uint64_t c = cost[cell];
    const uint32_t id = arg[cell];
    out[n].cost = c;
    out[n].cell = cell;
    out[n].arg = id;
    n++;
    if (c == kInf || id < w.move_base || id >= w.buf_id) break;
    if (id < w.tile_base) {
      if (!w.moves) break;
      uint32_t r = id - w.move_base;
      const uint32_t convert = r & 1u; r >>= 1;
      const uint32_t change = r % w.xw; r /= w.xw;
      const uint32_t dst = r % w.n_dst, op = r / w.n_dst;
      if (op >= 5 || !go(4 + op, dst)) break;
      if (change) {
        const int a = lay_axis[op];
        if (a < 0 || !go((uint32_t)a, x[a] ^ change)) break;
      }
      if (convert) {
        const int a = dt_axis[op];
        if (a < 0 || !go((uint32_t)a, 0)) break;
      }
    } else {
      if (!w.tiles) break;
      const uint32_t r = id - w.tile_base;
      if (!go(r / w.maxs, r % w.maxs)) break;
    }
  }
  *n_out = n;
}

hipError_t launch_chain(const ChainWalk& w, const uint64_t* cost, const uint16_t* arg, ChainEntry* out, uint32_t* n_out, hipStream_t st) {
  return launch_checked(chain_kernel, dim3(1), dim3(64), st, w, cost, arg, out, n_out);
}

__global__ __launch_bounds__(256) void zero_words_kernel(unsigned long long* p, uint32_t n) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < n) p[i] = 0;
}

void launch_zero_words(unsigned long long* p, uint32_t n, hipStream_t st) {
  if (n) hipLaunchKernelGGL(zero_words_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
}

}  // namespace mrl
