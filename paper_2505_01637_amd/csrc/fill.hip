// Rewrite evaluation + argmin over the Spec lattice.
//
// Paper, Section 4: a Spec's entry is the lowest-cost applicable rewrite, the
// rewrite's cost being the affine function of Section 3 of its sub-Specs'
// costs.  Here the table is filled bottom-up.
//
// An item is one shape (b,m,k,n) at one value of the passive level axis (the
// intermediate's level of a fused Spec; other kinds have one value): a set of
// entries closed under Moves.  A plan kernel decides, for every item and every
// value of the dtype bits, which level assignments fit their levels (most do
// not), as one bit mask per item (bit = level assignment in table order).  The
// whole table is set to (INF, NONE) by a launch of its own, beside the plan in
// large tables.  The rank is the sum of the operand levels.  A Move lowers the rank
// within an item, and a tile goes to the same level assignment of a shape of a
// lower dependency level, so the entries of one diagonal, level + rank, depend
// on earlier diagonals only.  The admissible level assignments are listed by
// diagonal, and one launch takes a diagonal: every candidate of an entry is a
// read of a finished entry, no workgroup waits for another, and nothing but
// the order of the launches has to be kept.
//
// Such a launch is bound by the chain of reads of one wave (unit, record, tile,
// sub-Spec) while the chip is not full, then by instruction issue, hence three
// forms of it: the reads of an entry shared out over several lanes; four
// entries that differ in their layouts only on four lanes, which share what
// does not depend on the layout; a lane per entry.
// Ties go to the lowest id: a lane meets its candidates in the order of their
// ids where it compares the cost alone, all else is compared by (cost, id).
// Nothing is reduced across workgroups: the table is deterministic.
//
// Large tables of which much fits are not filled by diagonals but a dependency
// level of shapes at a time (fill_shapes_kernel).
// Against the form it replaces (bundles of items in LDS, rank by rank with a
// barrier each, a launch per dependency level; 1,900 to 3,250 vector
// lane-instructions per entry), whole solves: two Matmuls composed 2742 ->
// 1960 us (16.8 M entries; G's fill 1.34 -> 0.79 ms), the vector-matrix product
// 668 -> 437, batched layouts 1061 -> 751, packed layouts 3058 -> 2404, the
// pipeline 3728 -> 3040.
#include <string.h>
#include <algorithm>
#include <hip/hip_runtime.h>
#include "compress.h"
#include "dev_params.h"

namespace mrl {

constexpr uint32_t kBatch = 8;         // tiles whose sub-Specs' costs are fetched together

struct Eval {
  uint64_t best;
  uint32_t arg;
  uint32_t n;
  uint32_t ovf;
};

// Keep the lexicographic minimum of (cost, rewrite id) among the candidates with ok set (all
// finite), so the evaluation order of the rewrites is free.  Written with selects: as branches
// the many calls cost more in exec-mask bookkeeping than the work they skip.
__device__ __forceinline__ void consider(Eval& e, uint64_t cand, uint32_t id, bool ok = true) {
  const bool better = ok & ((cand < e.best) | ((cand == e.best) & (id < e.arg)));
  e.best = better ? cand : e.best;
  e.arg = better ? id : e.arg;
}

// a * b for operands below 2^62 and 2^33; kLimit if the product reaches 2^62.
__device__ __forceinline__ uint64_t mul_or_limit(uint64_t a, uint64_t b) {
  const uint64_t lo = a * b;
  return (__umul64hi(a, b) != 0 || lo >= kLimit) ? kLimit : lo;
}

struct Shape {
  uint32_t si[4];
  uint64_t d[4];
  uint64_t numel[5];
};

__device__ __forceinline__ void load_shape(const DevParams* __restrict__ P, uint32_t shape, Shape& S) {
  uint32_t r = shape;
#pragma unroll
  for (int a = 0; a < 4; a++) {
    S.si[a] = r / P->shape_stride[a];
    r -= S.si[a] * P->shape_stride[a];
    S.d[a] = P->sizes[a][S.si[a]];
  }
  uint64_t b = S.d[0], m = S.d[1], k = S.d[2], n = S.d[3];
  if (P->kind == kKindM) { S.numel[0] = b * m * k; S.numel[1] = b * k * n; S.numel[2] = b * m * n; S.numel[3] = 0; S.numel[4] = 0; }
  else if (P->kind == kKindV) { S.numel[0] = m * n; S.numel[1] = m * n; S.numel[2] = 0; S.numel[3] = 0; S.numel[4] = 0; }
  else if (P->kind == kKindE) { S.numel[0] = m * n; S.numel[1] = n; S.numel[2] = m * n; S.numel[3] = 0; S.numel[4] = m * n; }   // [4]: the intermediate of a split
  else if (P->kind == kKindR) { S.numel[0] = m * n; S.numel[1] = m * n; S.numel[2] = 0; S.numel[3] = 0; S.numel[4] = 0; }
  else if (P->chain) { S.numel[0] = m * k; S.numel[1] = k * b; S.numel[2] = b * n; S.numel[3] = m * n; S.numel[4] = m * b; }   // b holds p
  else { S.numel[0] = m * k; S.numel[1] = k * n; S.numel[2] = n; S.numel[3] = m * n; S.numel[4] = m * n; }
}

// Shape part of microkernel j's predicate: number of repetitions, 0 if it fails
// (Section 2, Microkernel Selection; Figure 1 for BroadcastVecMultAdd).  The
// level/layout/dtype part is tabulated per entry (DevParams::mk_entry).
__device__ __forceinline__ uint64_t mk_shape_reps(const DevParams* __restrict__ P, const Shape& S, uint32_t j) {
  const uint32_t b = (uint32_t)S.d[0], m = (uint32_t)S.d[1], k = (uint32_t)S.d[2], n = (uint32_t)S.d[3];      // (a size is 32 bits, and so is its division)
  const uint32_t lanes = P->mk_lanes[j];
  switch (P->mk_kind[j]) {
    case 0: return (b == 1 && m == 1 && k == 1 && n == 1) ? 1 : 0;
    case 1: return (b == 1 && m == 1 && k == 1 && n % lanes == 0) ? n / lanes : 0;
    case 2: return (b == 1 && m == 1 && n == 1 && k % lanes == 0) ? k / lanes : 0;
    case 3: return (m == 1 && n == 1) ? 1 : 0;
    case 4: return (m == 1 && n % lanes == 0) ? n / lanes : 0;
    case 5: return (m == 1 && n == 1) ? 1 : 0;                       // Move Specs: m rows, n columns
    case 6:
    case 7: return (m == 1 && n % lanes == 0) ? n / lanes : 0;
    case 8:                                                          // bias add alone, ReLU alone: one element,
    case 10: return (m == 1 && n == 1) ? 1 : 0;
    case 9:                                                          // or one row of whole vectors
    case 11: return (m == 1 && n % lanes == 0) ? n / lanes : 0;
    default: return 0;
  }
}

__device__ __forceinline__ uint32_t lane_of(uint32_t v, uint32_t lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane); }

// ---------------------------------------------------------------- work lists
// The layouts a shape's tensors can have: operand i's layout field takes values below 1 << width(i)
// (the packed layouts need whole strips; an operand without a layout coordinate has width 0).
__device__ __forceinline__ uint32_t layout_width(const DevParams* __restrict__ P, const Shape& S, uint32_t i) {
  const uint32_t w = P->lay_w[i];
  if (!P->moves || w < 2) return w;
  const uint32_t cols = (uint32_t)(i == 0 ? S.d[2] : S.d[3]);
  return cols % P->strip == 0 ? 2u : 1u;
}

// What the fill needs of a shape, worked out once by the plan kernel.
struct alignas(16) ShapeRec {
  uint64_t numel[5];             // elements of the operands ([4]: the intermediate)
  uint32_t shape, si;            // index; the four size indices, a byte each
  uint32_t n_serial, n_tile;     // tile rewrites: serial loops, with parallel loops
  uint32_t tile_lo[4], tile_cnt; // first entry of each dimension's list of tiles, their numbers (a byte each)
  uint32_t mk_var;               // microkernels whose shape predicate holds (bits 0..7); packed layouts: layouts that exist << 8 (see variant_of)
};
static_assert(sizeof(ShapeRec) == 80, "read as five 16-byte pieces");

// Work lists.  A unit is an admissible (item, dtype bits, level assignment): the entries that differ in their layouts
// only (packed layouts: a part of these, see unit_parts).  Units are listed by diagonal, dependency level of the
// shape + rank of the level assignment: a Move lowers the rank within an item and a tile goes to the same level
// assignment of a shape of a lower level, so the units of one diagonal depend on earlier diagonals only.  Within a
// diagonal they lie level by level, then in the order of their items: neighbours share a shape and its tiles.
//
// plan: a lane per item, kBlockItems of one level to a block; writes the shapes' records, the items' masks (bit = level
// assignment in table order, one plane of nwp words per value of the dtype bits) and per block the units of every rank.
// scan: a workgroup per (level, rank) turns these into places within it, the last one to end adds up the diagonals.
// list: a lane per unit.  The whole list may be longer than its place in the scratch buffer:
// a window of it is written, as often as the host asks.  fit map: the bit map of the entries that fit, in table
// order (read by the compression), beside the fill.
// With a wave per shape, its lanes level assignments, the plan was bound by instruction issue (460 vector instructions a
// shape; a lane per item takes 9 per level assignment for 64 items): all sizes to 64 (262,144 shapes) 124 us and the list 61, now
// 31 and 46, the solve 1190 -> 1106.
constexpr uint32_t kBlockItems = 8;

// Level of block b: my_end = first block behind level `lane`.
__device__ __forceinline__ uint32_t level_of_block(uint32_t my_end, uint32_t b) { return (uint32_t)__popcll(__ballot(my_end <= b)); }

__global__ __launch_bounds__(256) void plan_kernel(const DevParams* __restrict__ P, const uint32_t* __restrict__ level_shapes, const uint32_t* __restrict__ level_off,
                                                   const uint32_t* __restrict__ blk_off, uint32_t n_levels, uint32_t n_blk, ShapeRec* __restrict__ recs,
                                                   unsigned long long* __restrict__ masks, uint32_t* __restrict__ cnt) {
  const uint32_t lane = threadIdx.x & 63u, b = (blockIdx.x * 256u + threadIdx.x) / kBlockItems, b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
  const uint32_t npass = P->npass, ncombo = P->ncombo, nwp = P->nwp, ndp = 1u << P->ndt, nw = ndp * nwp, NL = P->NL, nops = P->nops;
  __shared__ unsigned long long rank_masks[kMaxRanks][4];
  if (threadIdx.x < kMaxRanks * 4) rank_masks[threadIdx.x / 4][threadIdx.x % 4] = P->rank_mask[threadIdx.x / 4][threadIdx.x % 4];
  __syncthreads();
  const uint32_t my_end = lane < n_levels ? blk_off[lane + 1] : ~0u;
  uint32_t lev = 0;
#pragma unroll
  for (uint32_t k = 0; k < 64 / kBlockItems; k++) { const uint32_t l = level_of_block(my_end, b0 + k); lev = lane / kBlockItems == k ? l : lev; }
  uint32_t item = 0;
  bool have = b < n_blk;
  if (have) {
    item = level_off[lev] * npass + (b - blk_off[lev]) * kBlockItems + lane % kBlockItems;
    have = item < level_off[lev + 1] * npass;
  }
  unsigned long long m[4] = {0, 0, 0, 0};
  uint32_t parts = 0;
  if (have) {
    const uint32_t at = item / npass, pass = item - at * npass, shape = level_shapes[at];
    Shape S;
    load_shape(P, shape, S);
    uint32_t var = 0, nvb = 0;
    for (uint32_t i = nops; i-- > 0;) {         // from the lowest layout field up
      const uint32_t w = layout_width(P, S, i);
      if (i < 3) var |= w << (2 * i) | nvb << (8 + 4 * i);
      nvb += w;
    }
    if (P->moves) parts = nvb - P->unit_lay;
    if (pass == 0) {
      uint32_t n_serial = 0, n_par = 0, cnts = 0, mk = 0;
      uint32_t lo[4];
#pragma unroll
      for (int d = 0; d < 4; d++) {
        lo[d] = P->tile_off[d][S.si[d]];
        const uint32_t c = P->tile_off[d][S.si[d] + 1] - lo[d];
        cnts |= c << (8 * d);
        if (P->tile_dim_ok[d]) n_serial += c;
        if (P->par && d != 2) n_par += c;
      }
      for (uint32_t j = 0; j < P->nmk; j++) mk |= (mk_shape_reps(P, S, j) ? 1u : 0u) << j;
      ShapeRec r;
#pragma unroll
      for (int i = 0; i < 5; i++) r.numel[i] = S.numel[i];
      r.shape = shape; r.si = S.si[0] | S.si[1] << 8 | S.si[2] << 16 | S.si[3] << 24;
      r.n_serial = n_serial; r.n_tile = n_serial + n_par;
#pragma unroll
      for (int d = 0; d < 4; d++) r.tile_lo[d] = lo[d];
      r.tile_cnt = cnts;
      r.mk_var = mk | (P->moves ? (var & 0x3Fu) << 8 | (var >> 8 & 7u) << 14 | (var >> 12 & 7u) << 17 | (var >> 16 & 7u) << 20 | nvb << 23 : 0u);
      const uint4* from = reinterpret_cast<const uint4*>(&r);
      uint4* to = reinterpret_cast<uint4*>(recs + at);
#pragma unroll
      for (int i = 0; i < 5; i++) to[i] = from[i];
    }
    // ---- which level assignments fit ----
    const uint64_t mid = P->kind == kKindF ? S.numel[4] << 2 : 0;
    for (uint32_t dt = 0; dt < ndp; dt++) {
      // bit s of fit[l]: the operands of subset s together fit level l, next to the intermediate if it lives there
      uint64_t sum[16];
      sum[0] = 0;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const uint32_t bf = P->dt_bit[i] != kNoBit ? (dt >> P->dt_bit[i]) & 1u : P->base_bf16[i];
        const uint64_t bytes = (uint32_t)i < nops ? S.numel[i] << (bf ? 1u : 2u) : 0;
#pragma unroll
        for (int q = 0; q < 1 << i; q++) sum[q | 1 << i] = sum[q] + bytes;
      }
      uint32_t fit[4];
#pragma unroll
      for (uint32_t l = 0; l < 4; l++) {
        const uint64_t cap = P->cap[l], extra = l == pass ? mid : 0, room = cap - extra;
        uint32_t f = 0;
#pragma unroll
        for (int q = 0; q < 16; q++) f |= (sum[q] <= room ? 1u : 0u) << q;
        fit[l] = l >= NL ? 0xFFFFu : extra > cap ? 0u : f;
      }
      for (uint32_t w = 0; w < nwp; w++) {
        uint32_t half[2] = {0, 0};
#pragma unroll
        for (uint32_t h = 0; h < 2; h++) {
          const uint32_t c0 = w * 64 + h * 32, n = ncombo <= c0 ? 0u : ncombo - c0 < 32u ? ncombo - c0 : 32u;
          if (!n) break;
          uint32_t x = 0;
#pragma unroll
          for (uint32_t c = 0; c < 32; c++) {
            const uint32_t info = P->combo_info[c0 + c];      // (the same for all lanes)
            const uint32_t ok = fit[0] >> ((info >> 8) & 15u) & fit[1] >> ((info >> 12) & 15u) & fit[2] >> ((info >> 16) & 15u) & fit[3] >> ((info >> 20) & 15u);
            x = __builtin_amdgcn_alignbit(ok, x, 1);          // shifted in from above
          }
          half[h] = x & (n < 32u ? (1u << n) - 1u : ~0u);
        }
        const unsigned long long word = (unsigned long long)half[1] << 32 | half[0];
        masks[((size_t)shape * npass + pass) * nw + dt * nwp + w] = word;
        const uint32_t k = dt * nwp + w;
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) m[u] = u == k ? word : m[u];
      }
    }
  }
  for (uint32_t r = 0; r < P->nranks; r++) {
    uint32_t n = 0;
#pragma unroll
    for (uint32_t w = 0; w < 4; w++) n += (uint32_t)__popcll(m[w] & rank_masks[r][nwp > 1 ? w : 0]);      // (several words: no dtype bits)
    n <<= parts;
#pragma unroll
    for (uint32_t d = 1; d < kBlockItems; d <<= 1) n += (uint32_t)__shfl_xor((int)n, d, 64);
    if (b < n_blk && lane % kBlockItems == 0) cnt[(size_t)r * n_blk + b] = n;
  }
}

// seg: units of every (level, rank), then their first places in the list; host_diag: the diagonals' first places, and the
// end, straight to pinned host memory (behind a copy the next kernel would wait for it).
__global__ __launch_bounds__(1024) void scan_units_kernel(const uint32_t* __restrict__ blk_off, uint32_t n_levels, uint32_t n_ranks, uint32_t n_blk,
                                                          uint32_t* __restrict__ cnt, uint32_t* __restrict__ seg, uint32_t* __restrict__ host_diag, unsigned int* __restrict__ ticket) {
  __shared__ uint32_t sh[16];
  __shared__ uint32_t tot[kMaxLevels * kMaxRanks];
  __shared__ bool last;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, lev = blockIdx.x / n_ranks, r = blockIdx.x - lev * n_ranks;
  uint32_t* c = cnt + (size_t)r * n_blk;
  const uint32_t end = blk_off[lev + 1];
  uint32_t run = 0;
  for (uint32_t i0 = blk_off[lev]; i0 < end; i0 += 4096) {
    const uint32_t i = i0 + threadIdx.x * 4u;
    uint32_t v[4], mine = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) { v[k] = i + k < end ? c[i + k] : 0u; mine += v[k]; }
    uint32_t incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(incl, d, 64);
      if ((int)lane >= d) incl += o;
    }
    __syncthreads();
    if (lane == 63) sh[wave] = incl;
    __syncthreads();
    uint32_t before = run + incl - mine, total = 0;
#pragma unroll
    for (uint32_t w = 0; w < 16; w++) { const uint32_t x = sh[w]; before += w < wave ? x : 0u; total += x; }
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) { if (i + k < end) c[i + k] = before; before += v[k]; }
    run += total;
  }
  // (the totals pass between dies: written and read at the agent's scope, ordered by the ticket)
  if (threadIdx.x == 0) {
    __hip_atomic_store(seg + blockIdx.x, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1u == gridDim.x;
  }
  __syncthreads();
  if (!last) return;
  const uint32_t n_seg = n_levels * n_ranks;
  for (uint32_t i = threadIdx.x; i < n_seg; i += 1024) tot[i] = __hip_atomic_load(seg + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (wave) return;
  const uint32_t n_diag = n_levels + n_ranks - 1;       // lane d: diagonal d
  uint32_t n = 0;
  for (uint32_t l = 0; l < n_levels; l++) n += lane >= l && lane - l < n_ranks ? tot[l * n_ranks + lane - l] : 0u;
  uint32_t incl = n;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(incl, d, 64);
    if ((int)lane >= d) incl += o;
  }
  uint32_t at = incl - n;
  if (lane < n_diag) host_diag[lane] = at;
  if (lane == n_diag - 1) host_diag[n_diag] = seg[n_seg] = incl;
  for (uint32_t l = 0; l < n_levels; l++)
    if (lane >= l && lane - l < n_ranks) { seg[l * n_ranks + lane - l] = at; at += tot[l * n_ranks + lane - l]; }
}

// A unit of the list: x = index of its shape's record, y = pack (8 bits), dtype bits (2), level of the intermediate (2),
// part of its layouts (6), and from bit kUnitFit on, per operand and destination level, whether the level assignment with
// that operand there fits as well (its entries are finished, and only those are read).
constexpr uint32_t kUnitFit = 18;

// Units [w0, w0 + w_len) of the list: a workgroup per rank and n_items (at most kListItems) items, two of which a lane counts the units of;
// then a lane per unit looks up its item among the sums.  (A lane per rank and block of items that writes its units one after the
// other, as many as they are: 94 us for all sizes to 64, 335 for the pipeline; a lane per unit that searches the
// blocks' places in memory: 110 and 56.)
constexpr uint32_t kListItems = 512;
struct ListFirst { uint32_t block[kMaxRanks]; };       // first block that has units of the rank in the window
__global__ __launch_bounds__(256) void list_units_kernel(const DevParams* __restrict__ P, const uint32_t* __restrict__ level_shapes, const uint32_t* __restrict__ level_off,
                                                         const uint32_t* __restrict__ blk_off, uint32_t n_levels, uint32_t n_blk, const ShapeRec* __restrict__ recs,
                                                         const unsigned long long* __restrict__ masks, const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ seg,
                                                         uint2* __restrict__ list, uint32_t w0, uint32_t w_len, uint32_t n_items, uint32_t none_from, const ListFirst firsts) {
  const uint32_t n_units = seg[n_levels * P->nranks], b0 = firsts.block[blockIdx.y] + blockIdx.x * (n_items / kBlockItems);
  if (n_units >= none_from || b0 >= n_blk) return;
  if (n_units > w_len) {
    // a part of the list: nothing of these blocks may lie in it
    const uint32_t b1 = b0 + n_items / kBlockItems < n_blk ? b0 + n_items / kBlockItems : n_blk, r = blockIdx.y, n_ranks = P->nranks;
    uint32_t lev = 0;
    while (blk_off[lev + 1] <= b0) lev++;
    if (b1 <= blk_off[lev + 1]) {         // (of one level)
      const uint32_t start = seg[lev * n_ranks + r], from = start + cnt[(size_t)r * n_blk + b0];
      uint32_t to = ~0u;                  // behind a level's last block: the next level's units of the rank below, if it is not the diagonal's end
      if (b1 < blk_off[lev + 1]) to = start + cnt[(size_t)r * n_blk + b1];
      else if (lev + 1 < n_levels && r) to = seg[(lev + 1) * n_ranks + r - 1];
      if (to <= w0 || (from >= w0 && from - w0 >= w_len)) return;
    }
  }
  __shared__ uint32_t ends[kMaxLevels], waves[4], before[kListItems + 1], item_of[kListItems], to_of[kListItems / kBlockItems];
  __shared__ unsigned long long word_of[4][kListItems];
  __shared__ uint8_t parts_of[kListItems], packs[kMaxCombo];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, r = blockIdx.y;
  const uint32_t npass = P->npass, nwp = P->nwp, nw = nwp << P->ndt, n_ranks = P->nranks, nops = P->nops;
  if (tid < kMaxLevels) ends[tid] = tid < n_levels ? blk_off[tid + 1] : ~0u;
  packs[tid] = (uint8_t)P->combo_info[tid];
  unsigned long long rm[4];
#pragma unroll
  for (uint32_t w = 0; w < 4; w++) rm[w] = P->rank_mask[r][nwp > 1 ? w : 0];       // (several words: no dtype bits)
  __syncthreads();
  uint32_t n2[2] = {0, 0};
  {
    const uint32_t b = b0 + tid * 2u / kBlockItems;
    if (b < n_blk && tid * 2u < n_items) {
      uint32_t lev = 0;
#pragma unroll
      for (uint32_t d = kMaxLevels / 2; d > 0; d >>= 1) lev += ends[lev + d - 1] <= b ? d : 0u;      // levels that end at or before block b
      const uint32_t first = level_off[lev] * npass + (b - blk_off[lev]) * kBlockItems, end = level_off[lev + 1] * npass;
      if (tid * 2u % kBlockItems == 0) to_of[tid * 2u / kBlockItems] = seg[lev * n_ranks + r] + cnt[(size_t)r * n_blk + b] - w0;
#pragma unroll
      for (uint32_t q = 0; q < 2; q++) {
        const uint32_t j = tid * 2u + q, item = first + j % kBlockItems;
        if (item < end) {
          const uint32_t rec = item / npass, pass = item - rec * npass;
          const unsigned long long* mp = masks + ((size_t)level_shapes[rec] * npass + pass) * nw;
          const uint32_t parts = P->moves ? (recs[rec].mk_var >> 23) - P->unit_lay : 0u;
#pragma unroll
          for (uint32_t w = 0; w < 4; w++)
            if (w < nw) { const unsigned long long m = mp[w]; word_of[w][j] = m; n2[q] += (uint32_t)__popcll(m & rm[w]); }
          n2[q] <<= parts;
          item_of[j] = item;
          parts_of[j] = (uint8_t)parts;
        }
      }
    }
  }
  uint32_t incl = n2[0] + n2[1];
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(incl, d, 64);
    if ((int)lane >= d) incl += o;
  }
  if (lane == 63) waves[wave] = incl;
  __syncthreads();
  uint32_t at = incl - n2[0] - n2[1], total = 0;
#pragma unroll
  for (uint32_t w = 0; w < 4; w++) { const uint32_t x = waves[w]; at += w < wave ? x : 0u; total += x; }
  before[tid * 2u] = at;
  before[tid * 2u + 1] = at + n2[0];
  __syncthreads();
  uint32_t shift[4], step[4];
#pragma unroll
  for (uint32_t op = 0; op < 4; op++) { shift[op] = op < nops ? P->pack_shift[op] : 8u; step[op] = P->lvpow[op]; }      // (an operand that is not there: level 0)
  for (uint32_t u = tid; u < total; u += 256) {
    uint32_t j = 0;
#pragma unroll
    for (uint32_t d = kListItems / 2; d > 0; d >>= 1) j += before[j + d] <= u ? d : 0u;      // the last item that begins at or before it
    const uint32_t parts = parts_of[j], item = item_of[j], rec = item / npass, pass = item - rec * npass;
    uint32_t k = u - before[j];
    const uint32_t to = to_of[j / kBlockItems] + u - before[j / kBlockItems * kBlockItems], part = k & ((1u << parts) - 1u);
    if (to >= w_len) continue;            // (before the window: wraps around)
    k >>= parts;
    unsigned long long m[4];
#pragma unroll
    for (uint32_t w = 0; w < 4; w++) m[w] = w < nw ? word_of[w][j] : 0ull;
    uint32_t w = 0;
    unsigned long long x = m[0] & rm[0];
#pragma unroll
    for (uint32_t v = 1; v < 4; v++) {
      const uint32_t n = (uint32_t)__popcll(x);
      if (w == v - 1 && v < nw && k >= n) { k -= n; w = v; x = m[v] & rm[v]; }
    }
    const uint32_t dt = nwp > 1 ? 0u : w, combo = (nwp > 1 ? w * 64u : 0u) + nth_bit(x, k), pack = packs[combo];
    uint32_t y = pack | dt << 8 | pass << 10 | part << 12;
    const unsigned long long plane = w == 0 ? m[0] : w == 1 ? m[1] : w == 2 ? m[2] : m[3];
#pragma unroll
    for (uint32_t op = 0; op < 4; op++) {
      const uint32_t src = (pack >> shift[op]) & 3u;
#pragma unroll
      for (uint32_t dst = 0; dst < 3; dst++)
        if (dst < src) {
          const uint32_t c = combo - (src - dst) * step[op];
          unsigned long long word = plane;
          if (nwp > 1) {
            word = m[3];
            word = c < 192 ? m[2] : word;
            word = c < 128 ? m[1] : word;
            word = c < 64 ? m[0] : word;
          }
          y |= (uint32_t)(word >> (c & 63u) & 1ull) << (kUnitFit + op * 3 + dst);
        }
    }
    list[to] = make_uint2(rec, y);
  }
}

// The fit map, a word of 64 cells per lane, and two words of zeros behind it.
__global__ __launch_bounds__(256) void fit_map_kernel(const DevParams* __restrict__ P, uint32_t n_specs, const unsigned long long* __restrict__ masks, unsigned long long* __restrict__ map, uint32_t n_words) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n_words + 2) return;
  unsigned long long out = 0;
  if (i < n_words) {
    const uint32_t npass = P->npass, log2V = P->log2V, V = 1u << log2V, G = P->G, nwp = P->nwp, ndp = 1u << P->ndt, nw = nwp * ndp, nops = P->nops;
    uint32_t shape = (uint32_t)(((uint64_t)i * 64u) / G), off = i * 64u - shape * G, left = n_specs - i * 64u;
    left = left < 64u ? left : 64u;
    if (npass == 1 && !log2V) {                // a cell per level assignment: the masks one after the other
      for (uint32_t at = 0; at < left;) {
        const uint32_t room = 64u - (off & 63u), rest = G - off < left - at ? G - off : left - at, n = room < rest ? room : rest;
        const unsigned long long bits = masks[(size_t)shape * nw + (off >> 6)] >> (off & 63u) & (n >= 64u ? ~0ull : (1ull << n) - 1ull);
        out |= bits << at;
        at += n;
        off += n;
        if (off == G) { off = 0; shape++; }
      }
      map[i] = out;
      return;
    }
    // Four levels of the intermediate: 16 level assignments of one shape (256 to a shape), whose bits lie four apart.  (Cell by cell, as below: 93 us at
    // 113 M Specs, beside the fill, which it held up; now 11.)
    if (npass == 4 && !log2V) {
      const unsigned long long* mp = masks + (size_t)shape * 4u * nw + (off >> 8);
#pragma unroll
      for (uint32_t p = 0; p < 4; p++) {
        unsigned long long x = mp[p * nw] >> ((off >> 2) & 63u) & 0xFFFFull;
        x = (x | x << 24) & 0x000000FF000000FFull;
        x = (x | x << 12) & 0x000F000F000F000Full;
        x = (x | x << 6) & 0x0303030303030303ull;
        x = (x | x << 3) & 0x1111111111111111ull;
        out |= x << p;
      }
      map[i] = out;
      return;
    }
    uint32_t seen = ~0u;
    uint32_t combo = (off >> log2V) / npass, pass = (off >> log2V) - combo * npass;
    unsigned long long lays = 1;               // bit v: variant v (dtype bits 0) has layouts that exist
    for (uint32_t at = 0; at < left;) {
      if (shape != seen) {
        seen = shape;
        lays = 1;
        Shape S;
        if (P->moves) load_shape(P, shape, S);
        for (uint32_t j = nops; j-- > 0;) {    // from the lowest layout field up
          const uint32_t w = P->moves ? layout_width(P, S, j) : P->lay_w[j];
          if (!w) continue;
          const uint32_t step = 1u << P->lay_bit[j];
          lays |= lays << step;
          if (w == 2) lays |= lays << (2 * step);
        }
      }
      const uint32_t v0 = off & (V - 1u), n = V - v0 < left - at ? V - v0 : left - at;
      const unsigned long long* mp = masks + ((size_t)shape * npass + pass) * nw + (combo >> 6);
      unsigned long long bits = 0;
      for (uint32_t dt = 0; dt < ndp; dt++) bits |= (mp[dt * nwp] >> (combo & 63u) & 1ull) ? lays << dt : 0ull;
      bits = bits >> v0 & (n >= 64u ? ~0ull : (1ull << n) - 1ull);
      out |= bits << at;
      at += n;
      off += n;
      if (v0 + n == V && ++pass == npass) { pass = 0; combo++; }
      if (off == G) { off = 0; combo = 0; shape++; }
    }
  }
  map[i] = out;
}

// ---------------------------------------------------------------- one diagonal
// Variant of a unit's c-th entry.  Without packed layouts c is the layout bits; with them an item
// lists only the layouts that exist: var holds, per operand, the width of its field (2 bits at 2 * i)
// and the field's position inside c (3 bits at 6 + 3 * i).
template <bool MOVES>
__device__ __forceinline__ uint32_t variant_of(const FillArgs& A, uint32_t var, uint32_t c, uint32_t dt) {
  if (!MOVES) return c << A.ndt | dt;
  uint32_t v = dt;
#pragma unroll
  for (int i = 0; i < 3; i++) {
    const uint32_t w = (var >> (2 * i)) & 3u;
    if (w) v |= ((c >> ((var >> (6 + 3 * i)) & 7u)) & ((1u << w) - 1u)) << A.lay_bit[i];
  }
  return v;
}

// bufferize (FUSED): Matmul into the intermediate, then bias-add+ReLU out of it.  The composition
// of two Matmuls (Section 2.1): the first, (m, k, p), into the intermediate, then the second,
// (m, p, n), out of it; both are entries of the same Matmul table.  The bias-add + ReLU with its
// own bufferize: per level l in which the intermediate fits next to the operands that live there,
// the bias add into it plus the ReLU out of it.  si: the shape's size indices, a byte each; numel: its
// element counts.  Returns the number of candidates evaluated.
__device__ __forceinline__ uint32_t task_bufferize(const FillArgs& A, uint32_t si, const uint64_t* numel, uint32_t pack, uint32_t pass, uint32_t v, Eval& e) {
  const uint32_t NL = A.NL, i0 = si & 0xFFu, i1 = (si >> 8) & 0xFFu, i2 = (si >> 16) & 0xFFu, i3 = si >> 24;
  const auto level = [&](int i) { return (pack >> A.pack_shift[i]) & 3u; };
  const auto lay = [&](int i) { return A.lay_bit[i] != kNoBit ? (v >> A.lay_bit[i]) & 1u : 0u; };
  const auto at = [](uint32_t y, uint32_t bit) { return bit != kNoBit ? y << bit : 0u; };
  if (A.split) {
    const uint32_t rowM = (i1 * A.nsz3 + i3) * A.GM, rowE = (i1 * A.nsz3 + i3) * A.GE;
    const uint32_t l0 = level(0), l1 = level(1), l2 = level(2);
    const uint32_t va = at(lay(0), A.layM[0]), vr = at(lay(2), A.layE[1]);
    uint32_t cnt = 0;
    for (uint32_t l = 0; l < NL; l++) {
      const uint64_t bytes = 4u * (numel[2] + (l0 == l ? numel[0] : 0u) + (l1 == l ? numel[1] : 0u) + (l2 == l ? numel[2] : 0u));
      if (bytes > A.P->cap[l]) continue;
      const uint64_t ca = A.costM[rowM + ((l0 * NL + l1) * NL + l) * A.VM + va];
      const uint64_t cr = A.costE[rowE + (l * NL + l2) * A.VE + vr];
      if (ca != kInf && cr != kInf) {
        if (ca + cr >= kLimit) e.ovf = 1; else consider(e, ca + cr, A.buf_id + l);     // each below 2^62: no wrap
      }
      cnt++;
    }
    return cnt;
  }
  // (the composition's table has this lattice's p list for its k and n lists, and this lattice's k and n lists)
  const uint32_t rowM = (A.chain ? (i1 * A.nkM + i2) * A.nsz3 + i0 : (i1 * A.nkM + i2 + A.kM_first) * A.nsz3 + i3) * A.GM;
  const uint32_t rowE = A.chain ? ((i1 * A.nkM + i0) * A.nsz3 + i3) * A.GM : (i1 * A.nszE_n + i3) * A.GE;
  const uint32_t l0 = level(0), l1 = level(1), l2 = level(2), l3 = level(3);
  const uint32_t xm = ((l0 * NL + l1) * NL + pass) * A.VM + at(lay(0), A.layM[0]) + at(lay(1), A.layM[1]);
  const uint32_t xe = A.chain ? ((pass * NL + l2) * NL + l3) * A.VM + at(lay(2), A.layM[1]) + at(lay(3), A.layM[2])
                              : ((pass * NL + l2) * NL + l3) * A.VE + at(lay(3), A.layE[2]);
  const uint64_t* second = A.costE;
  if (A.chain) second = A.costM;
  const uint64_t cm = A.costM[rowM + xm], ce = second[rowE + xe];
  uint32_t zc = A.zero[3];             // (assignments: a conditional of members would select addresses, and copy them to scratch)
  if (pass == 2) zc = A.zero[2];
  if (pass == 1) zc = A.zero[1];
  if (pass == 0) zc = A.zero[0];
  const uint64_t z = mul_or_limit(zc, numel[4]);
  if (cm != kInf && ce != kInf) {
    const uint64_t sum = z + cm;          // each term <= 2^62: no wrap
    if (z >= kLimit || sum >= kLimit || sum + ce >= kLimit) e.ovf = 1; else consider(e, sum + ce, A.buf_id);
  }
  return 1;
}

// The best so far of one run of candidates in the order of their ids.
struct Best {
  uint64_t cost;
  uint32_t id;
  __device__ __forceinline__ void take(uint64_t cand, uint32_t cand_id, bool fin) {
    const bool better = fin && cand < cost;
    cost = better ? cand : cost;
    id = better ? cand_id : id;
  }
};

// The tiles of one entry, those of the dimensions one after the other, kBatch of them at a time in registers.
// MN: only m and n are tiled.  PAR: the parallel loops over b, m, n after the serial ones.
template <bool MN, bool PAR>
struct Tiles {
  uint32_t n, n_serial, done, q, at, b1, b2, b3, lo0, lo1, lo2, lo3;       // q: entry of the list behind tile `at`; b_d: the first tile of dimension d
  uint4 st[kBatch];
  __device__ __forceinline__ void begin(const uint32_t lo[4], uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
    b1 = c0; b2 = c0 + c1; b3 = b2 + c2; n = n_serial = b3 + c3;
    if (PAR) n += b2 + c3;
    lo0 = lo[0]; lo1 = lo[1]; lo2 = lo[2]; lo3 = lo[3];
    done = at = 0;
    q = MN ? lo1 : lo0;
    jump();
  }
  __device__ __forceinline__ void jump() {                  // (a dimension without tiles begins where the next one does)
    if (!MN) q = at == b1 ? lo1 : q;
    if (!MN) q = at == b2 ? lo2 : q;
    q = at == b3 ? lo3 : q;
    if (PAR) {
      q = at == n_serial ? lo0 : q;
      q = at == n_serial + b1 ? lo1 : q;
      q = at == n_serial + b2 ? lo3 : q;
    }
  }
  __device__ __forceinline__ void fetch(const TileStep* steps) {
#pragma unroll
    for (uint32_t u = 0; u < kBatch; u++) {
      if (at < n) st[u] = *(const uint4*)((const char*)steps + q * 16u);
      at++; q++;
      jump();
    }
  }
};

// Entry `cell` of a table; with SMALL its byte offset fits 32 bits.
template <bool SMALL>
__device__ __forceinline__ uint64_t at_cell(const uint64_t* table, uint32_t cell) {
  return SMALL ? *(const uint64_t*)((const char*)table + cell * 8u) : table[cell];
}

// The tiles of one entry, the first kBatch of them fetched: the same entry of a smaller shape; a parallel loop's body is an
// entry of the serial table.  over, over2: bits of finite candidates at 2^62 and above.
template <bool SMALL, bool MN, bool PAR>
__device__ __forceinline__ void take_tiles(const FillArgs& A, Tiles<MN, PAR>& tiles, uint32_t cell, Best& e, uint32_t& over, uint32_t& over2) {
  for (;;) {
    uint64_t sub[kBatch];
#pragma unroll
    for (uint32_t u = 0; u < kBatch; u++)
      if (tiles.done + u < tiles.n) {
        const uint64_t* table = A.cost;
        if (PAR && tiles.done + u >= tiles.n_serial) table = A.costM;
        sub[u] = at_cell<SMALL>(table, cell - tiles.st[u].x);
      }
#pragma unroll
    for (uint32_t u = 0; u < kBatch; u++)
      if (tiles.done + u < tiles.n) {
        const bool loop = PAR && tiles.done + u >= tiles.n_serial, fin = (uint32_t)(sub[u] >> 32) != ~0u;
        const uint32_t a = fin ? (loop ? tiles.st[u].w : tiles.st[u].y) : 0u;
        const uint64_t lo = (uint64_t)a * (uint32_t)sub[u] + (loop ? A.sync : A.s);   // (32 x 32 bits + 32 bits: no wrap)
        const uint64_t hi = (uint64_t)a * (uint32_t)(sub[u] >> 32) + (lo >> 32);      // bits 32.. of the sum
        over |= (uint32_t)hi;
        over2 |= (uint32_t)(hi >> 32);
        e.take((hi << 32) | (uint32_t)lo, tiles.st[u].z + (loop ? A.par_shift : 0u), fin);
      }
    tiles.done += kBatch;
    if (!__any(tiles.done < tiles.n)) break;
    tiles.fetch(A.steps);
  }
}

// One entry: a unit and one of its layouts.  Its candidates are read from finished entries of the table (and of the
// tables that it reads), several in flight.  Microkernels, Moves, the tiles of each dimension and the bufferize come in the
// order of their ids, so a strictly lower cost is all that has to be tested, but for converting Moves, whose ids lie
// between the others'.
// coef: DevParams::mcoef in LDS.  over, over2: bits of finite candidates at 2^62 and above.
// SMALL: coefficient * elements of every Move is below 2^62 and both fit 32 bits, and so do the table's byte offsets.
template <bool MOVES, bool SMALL, bool PAR, bool MN>
__device__ __forceinline__ void fill_entry(const FillArgs& A, const uint2 un, uint32_t c, const uint4* coef, uint32_t& n_rw, uint32_t& ovf) {
  const uint4* rp = reinterpret_cast<const uint4*>(A.recs) + (size_t)un.x * 5u;
  const uint4 r0 = rp[0], r1 = rp[1], r2 = rp[2], r3 = rp[3], r4 = rp[4];
  const uint32_t pack = un.y & 0xFFu, dt = (un.y >> 8) & 3u, pass = (un.y >> 10) & 3u, fit = un.y >> kUnitFit;
  const uint32_t log2V = A.log2V, nops = A.nops, NL = A.NL;
  const uint64_t numel[5] = {(uint64_t)r0.y << 32 | r0.x, (uint64_t)r0.w << 32 | r0.z, (uint64_t)r1.y << 32 | r1.x, (uint64_t)r1.w << 32 | r1.z, (uint64_t)r2.y << 32 | r2.x};
  const uint32_t shape = r2.z, si = r2.w, cnts = r4.z, mk_var = r4.w;
  const uint32_t tlo[4] = {r3.z, r3.w, r4.x, r4.y};
  uint32_t src[4], at = pass << log2V;
#pragma unroll
  for (uint32_t op = 0; op < 4; op++) {
    src[op] = op < nops ? (pack >> A.pack_shift[op]) & 3u : 0u;
    at += src[op] * A.mstride[op];
  }
  const uint32_t var = mk_var >> 8;
  if (MOVES) c |= ((un.y >> 12) & 63u) << A.unit_lay;
  const uint32_t v = variant_of<MOVES>(A, var, c, dt);
  const uint32_t cell = shape * A.G + (at | v);
  uint64_t* const cost = A.cost;

  // tiles, kBatch at a time; the first are requested before the Moves' entries
  const uint32_t c0 = cnts & 0xFFu, c1 = (cnts >> 8) & 0xFFu, c2 = (cnts >> 16) & 0xFFu, c3 = cnts >> 24;
  Tiles<MN, PAR> tiles;
  tiles.begin(tlo, MN ? 0u : c0, c1, MN ? 0u : c2, c3);
  if (!MOVES) tiles.fetch(A.steps);

  Best e{kInf, kNone};
  uint32_t over = 0, over2 = 0;
  // microkernels
  if (mk_var & 0xFFu) {
    for (uint32_t mm = A.mk_entry[(pack << log2V) + v] & mk_var & 0xFFu; mm; mm &= mm - 1) {
      const uint32_t m = (uint32_t)__ffs((int)mm) - 1u;
      Shape H;
#pragma unroll
      for (int d = 0; d < 4; d++) H.d[d] = A.P->sizes[d][(si >> (8 * d)) & 0xFFu];
      const uint64_t ck = mul_or_limit(A.P->mk_cost[m], mk_shape_reps(A.P, H, m));
      if (ck >= kLimit) ovf |= 1u;
      e.take(ck, m, ck < kLimit);
      n_rw++;
    }
  }

  // Moves
  if (!MOVES) {
    uint64_t sub[4][3][2];
#pragma unroll
    for (uint32_t op = 0; op < 4; op++) {
      if (op >= nops) break;
      const uint32_t lay = A.lay_xor[op], at0 = cell - src[op] * A.mstride[op];
#pragma unroll
      for (uint32_t dst = 0; dst < 3; dst++)
        if ((fit >> (op * 3 + dst)) & 1u) {
          const uint32_t to = at0 + dst * A.mstride[op];
          sub[op][dst][0] = at_cell<SMALL>(cost, to);
          if (lay) sub[op][dst][1] = at_cell<SMALL>(cost, to ^ lay);
        }
    }
#pragma unroll
    for (uint32_t op = 0; op < 4; op++) {
      if (op >= nops) break;
      const uint32_t lay = A.lay_xor[op];
      const uint4 ca = coef[op * 8 + src[op] * 2], cb = coef[op * 8 + src[op] * 2 + 1];
      const uint32_t cf[6] = {ca.x, ca.y, ca.z, ca.w, cb.x, cb.y};
      const uint32_t id0 = A.move_base + op * (NL - 1u) * 4u;
      const uint32_t cv_bit = A.cv_bit[op];                           // the dtype bit that a converting Move clears
      const bool cv_here = (dt & cv_bit) != 0;
      n_rw += cv_here ? 2u * cb.z : cb.z;                             // Moves that exist, whatever fits
      const auto price = [&](uint32_t k, uint32_t extra) {
        return SMALL ? (uint64_t)(k + extra) * (uint32_t)numel[op] : mul_or_limit((uint64_t)k + extra, numel[op]);
      };
#pragma unroll
      for (uint32_t dst = 0; dst < 3; dst++)
        if ((fit >> (op * 3 + dst)) & 1u) {
#pragma unroll
          for (uint32_t x = 0; x < 2; x++) {
            if (x && !lay) break;
            const uint64_t t = sub[op][dst][x];
            const uint32_t k = cf[dst * 2 + x];
            const bool fin = (uint32_t)(t >> 32) != ~0u && k != 0;    // 0: no such Move
            const uint64_t cand = t + price(k, 0);                    // each at most 2^62 when finite: no wrap
            over |= fin ? (uint32_t)(cand >> 32) : 0u;
            e.take(cand, id0 + dst * 4u + x * 2u, fin);
          }
        }
      if (cv_bit) {
        // to the type without the dtype bit; what does not fit there is (INF, NONE)
        Eval f;
        f.best = e.cost; f.arg = e.id;
        for (uint32_t dst = 0; dst < NL - 1u; dst++)
          for (uint32_t x = 0; x < (lay ? 2u : 1u); x++) {
            const uint32_t k = dst == 0 ? (x ? cf[1] : cf[0]) : dst == 1 ? (x ? cf[3] : cf[2]) : (x ? cf[5] : cf[4]);
            if (cv_here && dst < src[op] && k) {
              const uint64_t t = cost[((cell - (src[op] - dst) * A.mstride[op]) ^ (x ? lay : 0u)) & ~cv_bit];
              const bool fin = (uint32_t)(t >> 32) != ~0u;
              const uint64_t cand = t + price(k, A.convert);
              over |= fin ? (uint32_t)(cand >> 32) : 0u;
              consider(f, cand, id0 + dst * 4u + x * 2u + 1u, fin);
            }
          }
        e.cost = f.best; e.id = f.arg;
      }
    }
  } else {
    // priced by the table of alloc-bindings (bind_kernel); xw changes of layout, those that exist for this size
    const DevParams* __restrict__ P = A.P;
    const uint32_t yb = P->yb, xw = P->xw, per_op = 6u << (2 * yb), per_size = P->bind_d * per_op;
    const uint32_t i1 = (si >> 8) & 0xFFu, i2 = (si >> 16) & 0xFFu, i3 = si >> 24;
#pragma unroll
    for (uint32_t op = 0; op < 3; op++) {
      const uint32_t lw = P->lay_w[op], fw = (var >> (2 * op)) & 3u;
      const uint32_t y0 = fw ? (v >> A.lay_bit[op]) & ((1u << fw) - 1u) : 0u;
      const uint32_t dt_bit = P->dt_bit[op], bf = dt_bit != kNoBit ? (dt >> dt_bit) & 1u : P->base_bf16[op];
      const bool can_cv = A.cv_bit[op] != 0;
      const uint32_t rows = op == 1 ? i2 : i1, cols = op == 0 ? i2 : i3, s = src[op];
      const uint32_t id0 = A.move_base + op * (NL - 1u) * xw * 2u;
      n_rw += (s << lw) << (can_cv && bf ? 1u : 0u);
      for (uint32_t cv = 0; cv < (can_cv ? 2u : 1u); cv++) {
        const bool plane = !cv || bf;
        const uint32_t dc = P->bind_d == 3 && bf ? 1u + cv : 0u;
        const uint64_t* __restrict__ row = P->bind + ((size_t)(op == 2 ? P->nszV * P->nszV : 0u) + rows * P->nszV + cols) * per_size + dc * per_op + ((s * (s - 1u) / 2u) << (2 * yb)) + (y0 << yb);
        uint64_t b[3][4], t[3][4];
#pragma unroll
        for (uint32_t x = 0; x < 4; x++) {
          if (x >= (1u << lw)) break;
#pragma unroll
          for (uint32_t dst = 0; dst < 3; dst++) {
            // (a packed layout that this size cannot have: no such Spec.  Converted: what does not fit is (INF, NONE))
            const bool ok = plane && x < (1u << fw) && (cv ? dst < s : (fit >> (op * 3 + dst)) & 1u);
            b[dst][x] = t[dst][x] = kInf;
            if (ok) {
              b[dst][x] = row[(dst << (2 * yb)) + (y0 ^ x)];
              t[dst][x] = cost[((cell - (s - dst) * A.mstride[op]) ^ (x ? x << A.lay_bit[op] : 0u)) & ~(cv ? A.cv_bit[op] : 0u)];
            }
          }
        }
#pragma unroll
        for (uint32_t dst = 0; dst < 3; dst++)
#pragma unroll
          for (uint32_t x = 0; x < 4; x++) {
            if (x >= (1u << lw)) break;
            const bool fin = (uint32_t)(b[dst][x] >> 32) != ~0u && (uint32_t)(t[dst][x] >> 32) != ~0u;
            const uint64_t cand = t[dst][x] + b[dst][x];              // each at most 2^62 when finite: no wrap
            over |= fin ? (uint32_t)(cand >> 32) : 0u;
            const uint32_t id = id0 + (dst * xw + x) * 2u + cv;
            if (cv) { Eval f; f.best = e.cost; f.arg = e.id; consider(f, cand, id, fin); e.cost = f.best; e.id = f.arg; }
            else e.take(cand, id, fin);
          }
      }
    }
  }

  if (MOVES) tiles.fetch(A.steps);
  take_tiles<SMALL>(A, tiles, cell, e, over, over2);
  n_rw += r3.y;
  if (MN && !MOVES && A.has_buf) {
    Eval f;
    f.best = e.cost; f.arg = e.id; f.ovf = 0;
    n_rw += task_bufferize(A, si, numel, pack, pass, v, f);
    e.cost = f.best; e.id = f.arg;
    ovf |= f.ovf;
  }

  cost[cell] = e.cost;
  A.arg[cell] = (uint16_t)e.id;
  ovf |= (over >> 30) | over2;
}

// The least of (cost, id) over eight consecutive lanes (all of them active), in every one of them.
template <int CTRL>
__device__ __forceinline__ uint32_t lane_swap(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ void swap_min(Eval& e) {
  const uint32_t lo = lane_swap<CTRL>((uint32_t)e.best), hi = lane_swap<CTRL>((uint32_t)(e.best >> 32));
  const uint32_t id = lane_swap<CTRL>(e.arg);
  consider(e, (uint64_t)hi << 32 | lo, id);
}

// What a lane of a split entry needs of its operand, in LDS.
struct alignas(16) OpTab {
  uint32_t mstride, lay_xor, cv_bit, shift;        // shift: of the level inside the pack (unused operands: a place that is 0)
};

// The tiles that one of S lanes takes, B of them (S apart) at a time in registers; PAR: the parallel loops over b, m, n
// after the serial ones.
template <bool MN, bool PAR, uint32_t S, uint32_t B>
struct TileShare {
  uint32_t b1, b2, b3, n_serial, n, o0, o1, o2, o3;
  uint4 st[B];
  __device__ __forceinline__ TileShare(const uint4 r3, const uint4 r4, uint32_t cnts, bool active, uint32_t all) {
    const uint32_t c0 = MN ? 0u : cnts & 0xFFu, c1 = (cnts >> 8) & 0xFFu, c2 = MN ? 0u : (cnts >> 16) & 0xFFu;
    b1 = c0; b2 = b1 + c1; b3 = b2 + c2; n_serial = b3 + (cnts >> 24);
    n = active ? PAR ? all : n_serial : 0u;
    o0 = r3.z; o1 = r3.w - b1; o2 = r4.x - b2; o3 = r4.y - b3;
  }
  __device__ __forceinline__ void fetch(const TileStep* steps, uint32_t t0) {
    const uint32_t p0 = o0, p1 = o1, p2 = o2, p3 = o3, e1 = b1, e2 = b2, e3 = b3;       // (choosing among members would choose among addresses, and keep them in scratch)
#pragma unroll
    for (uint32_t u = 0; u < B; u++) {
      uint32_t t = t0 + u * S;
      if (t < n) {
        uint32_t o = p3;
        if (!MN) { o = t < e3 ? p2 : o; o = t < e2 ? p1 : o; o = t < e1 ? p0 : o; }
        else o = t < e3 ? p1 : o;
        if (PAR && t >= n_serial) {
          t -= n_serial;
          o = p3 + e3 - e2;
          o = t < e2 ? p1 : o;
          o = t < e1 ? p0 : o;
        }
        st[u] = *(const uint4*)((const char*)steps + (o + t) * 16u);
      }
    }
  }
};

// Four consecutive entries of a table.
struct Quad { uint64_t t[4]; };
constexpr uint64_t kNoCost = ~0ull >> 1;    // above every finite cost
template <bool SMALL>
__device__ __forceinline__ Quad quad_at(const uint64_t* table, uint32_t cell) {
  const uint4* p = SMALL ? reinterpret_cast<const uint4*>((const char*)table + cell * 8u) : reinterpret_cast<const uint4*>(table + cell);
  const uint4 a = p[0], b = p[1];
  return Quad{{(uint64_t)a.y << 32 | a.x, (uint64_t)a.w << 32 | a.z, (uint64_t)b.y << 32 | b.x, (uint64_t)b.w << 32 | b.z}};
}

// Four entries of one unit, which differ in its two lowest layout bits (and so lie next to each other: no dtype bits),
// shared by four lanes (all of them active): lane s takes the Moves of operand s and tiles s, s + 4, ....  What does not
// depend on the layout is worked out once for the four entries: the tiles and their places, the Moves and their prices;
// and an entry that a Move reads for one of the four with the layout kept serves another with it changed.
template <bool SMALL, bool PAR, bool MN>
__device__ __forceinline__ void fill_quad(const FillArgs& A, const uint2 un, uint32_t c, uint32_t s, bool active, const uint4* coef, const OpTab* tab, uint32_t& n_rw, uint32_t& ovf) {
  constexpr uint32_t kMine = 2;                       // tiles at a time
  const char* rec = (const char*)A.recs + (size_t)un.x * 80u;
  const uint4 r3 = reinterpret_cast<const uint4*>(rec)[3], r4 = reinterpret_cast<const uint4*>(rec)[4];
  const uint2 r2 = reinterpret_cast<const uint2*>(rec)[5];
  const uint64_t numel = reinterpret_cast<const uint64_t*>(rec)[s];
  const uint32_t pack = un.y & 0xFFu, pass = (un.y >> 10) & 3u, fit = un.y >> kUnitFit;
  const uint32_t log2V = A.log2V, nops = A.nops, NL = A.NL;
  const uint32_t shape = r2.x, si = r2.y, cnts = r4.z, mk_var = r4.w;
  uint32_t at = pass << log2V;
#pragma unroll
  for (uint32_t i = 0; i < 4; i++) if (i < nops) at += ((pack >> A.pack_shift[i]) & 3u) * A.mstride[i];
  const uint32_t cell = shape * A.G + (at | c);
  uint64_t* const cost = A.cost;
  const OpTab my = tab[s];
  const uint32_t src = s < nops ? (pack >> my.shift) & 3u : 0u;
  TileShare<MN, PAR, 4, kMine> tiles(r3, r4, cnts, active, r3.y);
  tiles.fetch(A.steps, s);

  Best e[4];
#pragma unroll
  for (int r = 0; r < 4; r++) e[r] = Best{kNoCost, kNone};
  uint32_t over = 0, over2 = 0;
  // Moves: an entry that is not finite reads as 2^63 - 1, so with any price added it has bit 63 set and is above kNoCost
  {
    const uint32_t my_fit = active ? (fit >> (3u * s)) & 7u : 0u, at0 = cell - src * my.mstride, lay = my.lay_xor, id0 = A.move_base + s * (NL - 1u) * 4u;
    Quad q[3], x[3];
#pragma unroll
    for (uint32_t dst = 0; dst < 3; dst++)
      if ((my_fit >> dst) & 1u) {
        q[dst] = quad_at<SMALL>(cost, at0 + dst * my.mstride);
        if (lay >= 4) x[dst] = quad_at<SMALL>(cost, (at0 + dst * my.mstride) ^ lay);
      }
    const uint4 ca = coef[s * 8 + src * 2], cb = coef[s * 8 + src * 2 + 1];
    const uint32_t cf[6] = {ca.x, ca.y, ca.z, ca.w, cb.x, cb.y};
    if (active) n_rw += 4u * cb.z;                                  // Moves that exist, whatever fits
    const auto add = [&](const Quad& t, uint32_t k, uint32_t id) {
      // no such Move: a price of 2^63
      const uint64_t price = SMALL ? (uint64_t)k * (uint32_t)numel : mul_or_limit(k, numel), b = k ? price : 1ull << 63;
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const uint64_t cand = (t.t[r] & kNoCost) + b;
        over = (int32_t)(cand >> 32) > (int32_t)over ? (uint32_t)(cand >> 32) : over;
        e[r].take(cand, id, true);
      }
    };
#pragma unroll
    for (uint32_t dst = 0; dst < 3; dst++)
      if ((my_fit >> dst) & 1u) {
        add(q[dst], cf[dst * 2], id0 + dst * 4u);
        if (lay) {
          if (lay < 4) {
            const bool one = lay == 1;
            x[dst] = Quad{{one ? q[dst].t[1] : q[dst].t[2], one ? q[dst].t[0] : q[dst].t[3], one ? q[dst].t[3] : q[dst].t[0], one ? q[dst].t[2] : q[dst].t[1]}};
          }
          add(x[dst], cf[dst * 2 + 1], id0 + dst * 4u + 2u);
        }
      }
  }

  // tiles: the same entries of a smaller shape; a parallel loop's body: entries of the serial table
  for (uint32_t t0 = s; __any(t0 < tiles.n); t0 += kMine * 4u) {
    if (t0 != s) tiles.fetch(A.steps, t0);
    Quad sub[kMine];
#pragma unroll
    for (uint32_t u = 0; u < kMine; u++)
      if (t0 + u * 4u < tiles.n) {
        const uint64_t* table = cost;
        if (PAR && t0 + u * 4u >= tiles.n_serial) table = A.costM;
        sub[u] = quad_at<SMALL>(table, cell - tiles.st[u].x);
      }
#pragma unroll
    for (uint32_t u = 0; u < kMine; u++)
      if (t0 + u * 4u < tiles.n) {
        const bool loop = PAR && t0 + u * 4u >= tiles.n_serial;
        const uint32_t trips = loop ? tiles.st[u].w : tiles.st[u].y, more = loop ? A.sync : A.s, id = tiles.st[u].z + (loop ? A.par_shift : 0u);
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const uint64_t t = sub[u].t[r];
          const bool fin = (uint32_t)(t >> 32) != ~0u;
          const uint32_t a = fin ? trips : 0u;
          const uint64_t lo = (uint64_t)a * (uint32_t)t + more;                         // (32 x 32 bits + 32 bits: no wrap)
          const uint64_t hi = (uint64_t)a * (uint32_t)(t >> 32) + (lo >> 32);           // bits 32.. of the sum
          over2 |= (uint32_t)hi >> 30 | (uint32_t)(hi >> 32);
          e[r].take((hi << 32) | (uint32_t)lo, id, fin);
        }
      }
  }
  if (s == 0 && active) n_rw += 4u * r3.y;
  if (active && ((mk_var & 0xFFu) | (MN ? A.has_buf : 0u))) {
    // microkernels and the bufferize: lane s for entry s
    Eval f;
    f.best = kInf; f.arg = kNone; f.ovf = 0;
    if (mk_var & 0xFFu) {
      for (uint32_t mm = A.mk_entry[(pack << log2V) + c + s] & mk_var & 0xFFu; mm; mm &= mm - 1) {
        const uint32_t m = (uint32_t)__ffs((int)mm) - 1u;
        Shape H;
#pragma unroll
        for (int d = 0; d < 4; d++) H.d[d] = A.P->sizes[d][(si >> (8 * d)) & 0xFFu];
        const uint64_t ck = mul_or_limit(A.P->mk_cost[m], mk_shape_reps(A.P, H, m));
        if (ck >= kLimit) f.ovf = 1; else consider(f, ck, m);
        n_rw++;
      }
    }
    if (MN && A.has_buf) {
      const uint64_t* np = reinterpret_cast<const uint64_t*>(rec);
      const uint64_t all[5] = {np[0], np[1], np[2], np[3], np[4]};
      n_rw += task_bufferize(A, si, all, pack, pass, c + s, f);
    }
    ovf |= f.ovf;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      Eval g;
      g.best = e[r].cost; g.arg = e[r].id;
      consider(g, f.best, f.arg, s == (uint32_t)r && f.best != kInf);
      e[r].cost = g.best; e[r].id = g.arg;
    }
  }
  // the least of the four lanes: lane s keeps entry s
  Eval best;
  best.best = kInf; best.arg = kNone;
#pragma unroll
  for (int r = 0; r < 4; r++) {
    Eval g;
    g.best = e[r].cost; g.arg = e[r].id;
    swap_min<0xB1>(g);                     // lanes ^ 1
    swap_min<0x4E>(g);                     // lanes ^ 2
    best.best = s == (uint32_t)r ? g.best : best.best;
    best.arg = s == (uint32_t)r ? g.arg : best.arg;
  }
  if (active) {
    cost[cell + s] = best.arg == kNone ? kInf : best.best;
    A.arg[cell + s] = (uint16_t)best.arg;
  }
  ovf |= ((int32_t)over >= (1 << 30) ? 1u : 0u) | over2;
}

// One entry shared by S lanes (all of them active), eight or, without layouts, four: lane s takes the Moves of operand s & 3
// that change the layout by s >> 2 (or s >> 2 + 2), and tiles s, s + S, ...; the first also the microkernels and the
// bufferize.
constexpr uint32_t lg_split_lanes(bool lay) { return lay ? 3u : 2u; }
constexpr uint32_t split_lanes(bool lay) { return 1u << lg_split_lanes(lay); }
template <bool LAY, bool MOVES, bool SMALL, bool PAR, bool MN>
__device__ __forceinline__ void fill_entry_split(const FillArgs& A, const uint2 un, uint32_t c, uint32_t s, bool active, const uint4* coef, const OpTab* tab, uint32_t& n_rw, uint32_t& ovf) {
  constexpr uint32_t kMine = 4, S = split_lanes(LAY); // tiles at a time
  const uint32_t op = s & 3u, x0 = s >> 2;
  const char* rec = (const char*)A.recs + (size_t)un.x * 80u;
  const uint4 r3 = reinterpret_cast<const uint4*>(rec)[3], r4 = reinterpret_cast<const uint4*>(rec)[4];
  const uint2 r2 = reinterpret_cast<const uint2*>(rec)[5];
  const uint64_t numel = reinterpret_cast<const uint64_t*>(rec)[op];
  const uint32_t pack = un.y & 0xFFu, dt = (un.y >> 8) & 3u, pass = (un.y >> 10) & 3u, fit = un.y >> kUnitFit;
  const uint32_t log2V = A.log2V, nops = A.nops, NL = A.NL;
  const uint32_t shape = r2.x, si = r2.y, cnts = r4.z, mk_var = r4.w;
  uint32_t at = pass << log2V;
#pragma unroll
  for (uint32_t i = 0; i < 4; i++) if (i < nops) at += ((pack >> A.pack_shift[i]) & 3u) * A.mstride[i];
  const uint32_t var = mk_var >> 8;
  if (MOVES) c |= ((un.y >> 12) & 63u) << A.unit_lay;
  const uint32_t v = variant_of<MOVES>(A, var, c, dt);
  const uint32_t cell = shape * A.G + (at | v);
  uint64_t* const cost = A.cost;
  const OpTab my = tab[op];
  const uint32_t src = op < nops && active ? (pack >> my.shift) & 3u : 0u;

  TileShare<MN, PAR, S, kMine> tiles(r3, r4, cnts, active, r3.y);
  tiles.fetch(A.steps, s);

  Eval e;
  e.best = kInf; e.arg = kNone; e.ovf = 0;
  uint32_t over = 0, over2 = 0;
  const auto add = [&](uint64_t t, uint64_t b, uint32_t id, bool ok) {        // each at most 2^62 when finite: no wrap
    const bool fin = ok && (uint32_t)(t >> 32) != ~0u;
    const uint64_t cand = t + b;
    over |= fin ? (uint32_t)(cand >> 32) : 0u;
    consider(e, cand, id, fin);
  };
  // Moves
  const uint32_t my_fit = active ? (fit >> (3u * op)) & 7u : 0u, at0 = cell - src * my.mstride;
  if (!MOVES) {
    const bool part = x0 == 0 || (LAY && my.lay_xor != 0);
    uint64_t sub[3];
#pragma unroll
    for (uint32_t dst = 0; dst < 3; dst++)
      if (part && ((my_fit >> dst) & 1u)) sub[dst] = at_cell<SMALL>(cost, (at0 + dst * my.mstride) ^ (x0 ? my.lay_xor : 0u));
    const uint4 ca = coef[op * 8 + src * 2], cb = coef[op * 8 + src * 2 + 1];
    const uint32_t k[3] = {x0 ? ca.y : ca.x, x0 ? ca.w : ca.z, x0 ? cb.y : cb.x};
    const uint32_t id0 = A.move_base + op * (NL - 1u) * 4u + x0 * 2u;
    const bool cv_here = (dt & my.cv_bit) != 0;
    if (x0 == 0 && src) n_rw += cv_here ? 2u * cb.z : cb.z;             // Moves that exist, whatever fits
    const auto price = [&](uint32_t kk, uint32_t extra) { return SMALL ? (uint64_t)(kk + extra) * (uint32_t)numel : mul_or_limit((uint64_t)kk + extra, numel); };
#pragma unroll
    for (uint32_t dst = 0; dst < 3; dst++)
      if (part && ((my_fit >> dst) & 1u)) add(sub[dst], price(k[dst], 0), id0 + dst * 4u, k[dst] != 0);
    if (__any(cv_here)) {
      // to the type without the dtype bit; what does not fit there is (INF, NONE)
#pragma unroll
      for (uint32_t dst = 0; dst < 3; dst++)
        if (part && cv_here && dst < src && k[dst])
          add(at_cell<SMALL>(cost, ((at0 + dst * my.mstride) ^ (x0 ? my.lay_xor : 0u)) & ~my.cv_bit), price(k[dst], A.convert), id0 + dst * 4u + 1u, true);
    }
  } else if (op < 3) {
    const DevParams* __restrict__ P = A.P;
    const uint32_t yb = P->yb, xw = P->xw, per_op = 6u << (2 * yb), per_size = P->bind_d * per_op;
    const uint32_t i1 = (si >> 8) & 0xFFu, i2 = (si >> 16) & 0xFFu, i3 = si >> 24;
    const uint32_t lw = P->lay_w[op], lb = P->lay_bit[op], fw = (var >> (2 * op)) & 3u, y0 = fw ? (v >> lb) & ((1u << fw) - 1u) : 0u;
    const uint32_t dt_bit = P->dt_bit[op], bf = dt_bit != kNoBit ? (dt >> dt_bit) & 1u : P->base_bf16[op];
    const uint32_t rows = op == 1 ? i2 : i1, cols = op == 0 ? i2 : i3;
    const uint32_t id0 = A.move_base + op * (NL - 1u) * xw * 2u;
    if (x0 == 0) n_rw += (src << lw) << (my.cv_bit && bf ? 1u : 0u);
    for (uint32_t cv = 0; cv < 2; cv++) {
      if (cv && !__any(my.cv_bit && bf)) break;
      const bool plane = !cv || (my.cv_bit && bf);
      const uint32_t dc = P->bind_d == 3 && bf ? 1u + cv : 0u;
      const uint64_t* __restrict__ row = P->bind + ((size_t)(op == 2 ? P->nszV * P->nszV : 0u) + rows * P->nszV + cols) * per_size + dc * per_op + ((src * (src - 1u) / 2u) << (2 * yb)) + (y0 << yb);
      uint64_t b[3][2], t[3][2];
#pragma unroll
      for (uint32_t u = 0; u < 2; u++) {
        const uint32_t x = x0 + 2u * u;
#pragma unroll
        for (uint32_t dst = 0; dst < 3; dst++) {
          // (a packed layout that this size cannot have: no such Spec.  Converted: what does not fit is (INF, NONE))
          const bool ok = plane && x < (1u << fw) && (cv ? dst < src : (my_fit >> dst) & 1u);
          b[dst][u] = t[dst][u] = kInf;
          if (ok) {
            b[dst][u] = row[(dst << (2 * yb)) + (y0 ^ x)];
            t[dst][u] = cost[((at0 + dst * my.mstride) ^ (x ? x << lb : 0u)) & ~(cv ? my.cv_bit : 0u)];
          }
        }
      }
#pragma unroll
      for (uint32_t dst = 0; dst < 3; dst++)
#pragma unroll
        for (uint32_t u = 0; u < 2; u++) add(t[dst][u], b[dst][u], id0 + (dst * xw + x0 + 2u * u) * 2u + cv, (uint32_t)(b[dst][u] >> 32) != ~0u);
    }
  }

  // tiles: the same entry of a smaller shape; a parallel loop's body is an entry of the serial table
  for (uint32_t t0 = s; __any(t0 < tiles.n); t0 += kMine * S) {
    if (t0 != s) tiles.fetch(A.steps, t0);
    uint64_t sub[kMine];
#pragma unroll
    for (uint32_t u = 0; u < kMine; u++)
      if (t0 + u * S < tiles.n) {
        const uint64_t* table = cost;
        if (PAR && t0 + u * S >= tiles.n_serial) table = A.costM;
        sub[u] = at_cell<SMALL>(table, cell - tiles.st[u].x);
      }
#pragma unroll
    for (uint32_t u = 0; u < kMine; u++)
      if (t0 + u * S < tiles.n) {
        const bool loop = PAR && t0 + u * S >= tiles.n_serial, fin = (uint32_t)(sub[u] >> 32) != ~0u;
        const uint32_t a = fin ? (loop ? tiles.st[u].w : tiles.st[u].y) : 0u;
        const uint64_t lo = (uint64_t)a * (uint32_t)sub[u] + (loop ? A.sync : A.s);
        const uint64_t hi = (uint64_t)a * (uint32_t)(sub[u] >> 32) + (lo >> 32);      // bits 32.. of the sum
        over |= (uint32_t)hi;
        over2 |= (uint32_t)(hi >> 32);
        consider(e, (hi << 32) | (uint32_t)lo, tiles.st[u].z + (loop ? A.par_shift : 0u), fin);
      }
  }
  if (s == 0 && active) {
    n_rw += r3.y;                          // serial and parallel loops
    if (mk_var & 0xFFu) {
      for (uint32_t mm = A.mk_entry[(pack << log2V) + v] & mk_var & 0xFFu; mm; mm &= mm - 1) {
        const uint32_t m = (uint32_t)__ffs((int)mm) - 1u;
        Shape H;
#pragma unroll
        for (int d = 0; d < 4; d++) H.d[d] = A.P->sizes[d][(si >> (8 * d)) & 0xFFu];
        const uint64_t ck = mul_or_limit(A.P->mk_cost[m], mk_shape_reps(A.P, H, m));
        if (ck >= kLimit) ovf |= 1u; else consider(e, ck, m);
        n_rw++;
      }
    }
    if (MN && !MOVES && A.has_buf) {
      const uint64_t* np = reinterpret_cast<const uint64_t*>(rec);
      const uint64_t all[5] = {np[0], np[1], np[2], np[3], np[4]};
      n_rw += task_bufferize(A, si, all, pack, pass, v, e);
    }
  }
  swap_min<0xB1>(e);                       // lanes ^ 1
  swap_min<0x4E>(e);                       // lanes ^ 2
  if (S == 8) swap_min<0x141>(e);          // the other four of eight (mirrored: the lanes of four agree by now)
  if (s == 0 && active) {
    cost[cell] = e.best;
    A.arg[cell] = (uint16_t)e.arg;
  }
  ovf |= e.ovf | (over >> 30) | over2;
}

// (rewrites evaluated: the only sums over workgroups)
__device__ __forceinline__ void flush_counters(Counters* __restrict__ ctr, uint32_t n_rw, uint32_t ovf) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) n_rw += __shfl_down(n_rw, d, 64);
  if ((threadIdx.x & 63u) == 0 && n_rw) atomicAdd(&ctr->n_rewrites[blockIdx.x % kCtrSlots], (unsigned long long)n_rw);
  if (ovf) atomicOr(&ctr->overflow, 1u);
}

// The operands' constants to LDS, and the Move coefficients.
__device__ __forceinline__ void load_tabs(const FillArgs& A, uint4* coef, OpTab* tab) {
  if (threadIdx.x < 32) coef[threadIdx.x] = reinterpret_cast<const uint4*>(A.P->mcoef)[threadIdx.x];
  if (threadIdx.x < 4) {
    const DevParams* P = A.P;
    const uint32_t i = threadIdx.x;
    tab[i] = OpTab{P->mstride[i], i < A.nops && P->lay_bit[i] != kNoBit ? 1u << P->lay_bit[i] : 0u, P->can_convert[i] && P->dt_bit[i] != kNoBit ? 1u << P->dt_bit[i] : 0u, P->pack_shift[i]};
  }
  __syncthreads();
}

// Workgroups go to the dies in turn: this one's place where each die has a stretch of consecutive ones (neighbours share
// units' records, children and lines of the table, and a die has an L2 of its own).
constexpr uint32_t kDies = 8;
__device__ __forceinline__ uint32_t die_block() {
  const uint32_t n = gridDim.x, x = blockIdx.x % kDies, full = n / kDies, more = n % kDies;
  return x * full + (x < more ? x : more) + blockIdx.x / kDies;
}

// A diagonal: a lane per entry, the layouts of a unit in consecutive lanes (1 << unit_lay of them).
template <bool MOVES, bool SMALL, bool PAR, bool MN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void fill_entry_kernel(const FillArgs A, const uint2* __restrict__ units, uint32_t n_units) {
  __shared__ uint4 coef[32];
  __shared__ OpTab tab[4];
  const uint64_t t = (uint64_t)die_block() * 256u + threadIdx.x;
  const uint32_t u = (uint32_t)(t >> A.unit_lay);
  const uint2 un = units[u < n_units ? u : 0u];
  load_tabs(A, coef, tab);
  uint32_t n_rw = 0, ovf = 0;
  if (u < n_units) fill_entry<MOVES, SMALL, PAR, MN>(A, un, (uint32_t)t & ((1u << A.unit_lay) - 1u), coef, n_rw, ovf);
  flush_counters(A.ctr, n_rw, ovf);
}

// Four lanes per four entries (the lattice has two layout bits and more, and no dtype bits).
template <bool SMALL, bool PAR, bool MN>
__global__ __launch_bounds__(256) void fill_quad_kernel(const FillArgs A, const uint2* __restrict__ units, uint32_t n_units) {
  __shared__ uint4 coef[32];
  __shared__ OpTab tab[4];
  const uint64_t t = (uint64_t)die_block() * 256u + threadIdx.x;
  const uint32_t u = (uint32_t)(t >> A.unit_lay);
  const uint2 un = units[u < n_units ? u : 0u];
  load_tabs(A, coef, tab);
  uint32_t n_rw = 0, ovf = 0;
  fill_quad<SMALL, PAR, MN>(A, un, (uint32_t)t & ((1u << A.unit_lay) - 4u), (uint32_t)t & 3u, u < n_units, coef, tab, n_rw, ovf);
  flush_counters(A.ctr, n_rw, ovf);
}

// Eight lanes per entry, or four without layouts.
template <bool LAY, bool MOVES, bool SMALL, bool PAR, bool MN>
__global__ __launch_bounds__(256) void fill_split_kernel(const FillArgs A, const uint2* __restrict__ units, uint32_t n_units) {
  constexpr uint32_t lgS = lg_split_lanes(LAY);
  __shared__ uint4 coef[32];
  __shared__ OpTab tab[4];
  const uint64_t t = ((uint64_t)die_block() * 256u + threadIdx.x) >> lgS;
  const uint32_t u = (uint32_t)(t >> A.unit_lay);
  const uint2 un = units[u < n_units ? u : 0u];
  load_tabs(A, coef, tab);
  uint32_t n_rw = 0, ovf = 0;
  fill_entry_split<LAY, MOVES, SMALL, PAR, MN>(A, un, (uint32_t)t & ((1u << A.unit_lay) - 1u), threadIdx.x & ((1u << lgS) - 1u), u < n_units, coef, tab, n_rw, ovf);
  flush_counters(A.ctr, n_rw, ovf);
}

// Several small diagonals one after the other, in one workgroup: its waves share a compute unit and so its L1, and a
// barrier orders what they write and read.  Only those that the workgroup takes in one go: with up to 2048 entries in a chain one
// compute unit's instruction issue is the bound (the vector-matrix product 473 -> 919 us; no chain at all: 485).
template <bool LAY, bool MOVES, bool SMALL, bool PAR, bool MN>
__global__ __launch_bounds__(kChainThreads) void fill_chain_kernel(const FillArgs A, const uint2* __restrict__ units, const DiagRun run) {
  __shared__ uint4 coef[32];
  __shared__ OpTab tab[4];
  constexpr uint32_t lgS = lg_split_lanes(LAY);
  load_tabs(A, coef, tab);
  uint32_t n_rw = 0, ovf = 0;
  for (uint32_t d = 0; d < run.n; d++) {
    const uint32_t first = run.start[d], tasks = (run.start[d + 1] - first) << A.unit_lay;
    for (uint32_t t0 = 0; t0 < tasks; t0 += kChainThreads >> lgS) {
      const uint32_t t = t0 + (threadIdx.x >> lgS);
      if (__all(t >= tasks)) break;
      fill_entry_split<LAY, MOVES, SMALL, PAR, MN>(A, units[first + (t < tasks ? t >> A.unit_lay : 0u)], t & ((1u << A.unit_lay) - 1u), threadIdx.x & ((1u << lgS) - 1u), t < tasks, coef, tab, n_rw, ovf);
    }
    __syncthreads();
  }
  flush_counters(A.ctr, n_rw, ovf);
}

// ---------------------------------------------------------------- a dependency level of shapes at once
// A diagonal takes a twelfth or so of a shape's entries, which lie all over its group: where most of them fit, every line of the group,
// and of the groups that its tiles lead to, is read again for almost every rank.  Large tables of which much fits, and whose groups are small (no layouts, or a
// Matmul's), are bound by that (all sizes to 64, everything fits: 49 M lines missed in the L2s, the fill 1.83 ms).  So here a workgroup takes whole groups, a launch
// a dependency level of shapes: first a lane per cell takes the tiles, one line after the other, with the list of tiles in scalar registers; then the Moves, inside the
// group, which stays in LDS, rank by rank: a few lanes per item, which no other wave touches, so that no barrier is needed between two
// ranks.  8.6 M lines missed, 0.75 ms of kernels (the bundles of items that the diagonals replaced: 1.29); bound by instruction issue, the ranks' the larger part.
// The rule is at by_shapes_from.
constexpr uint32_t kLgShapeCells = 10, kShapeCells = 1u << kLgShapeCells;       // of a workgroup, a quarter of them a wave's
constexpr uint32_t kShapeBatch = 8;          // tiles whose costs are fetched together
constexpr uint64_t kShapeUnits = 1u << 20;   // a table of fewer is never taken this way
constexpr uint32_t kNotHere = 1u << 16;      // id of a cell that does not fit
struct RankOff { uint16_t at[kMaxRanks + 2]; };                                  // DevParams::rank_off

// A group has 1 << lg_cells places (a wave's 64 cells are of one shape), an item 1 << lg_lanes lanes.
template <bool LAY, bool SMALL, bool PAR, bool MN>
__global__ __launch_bounds__(256) void fill_shapes_kernel(const FillArgs A, const RankOff ranks, const ShapeRec* __restrict__ all_recs, const TileStep* __restrict__ steps,
                                                          const unsigned long long* __restrict__ masks, uint32_t first, uint32_t n_shapes, uint32_t lg_cells, uint32_t lg_lanes) {
  constexpr uint32_t kChanges = LAY ? 2u : 1u;
  __shared__ uint32_t coef[128];                                  // DevParams::mcoef
  __shared__ uint64_t costs[kShapeCells];
  // of the Moves, [shape][operand][source level][layout kept, changed][destination]: 2^63 where there is none; in the place of destination 3:
  // how many there are (64 cells and more to a shape, with layouts 128: by_shapes_from)
  __shared__ uint64_t prices[kShapeCells / 4][4];
  __shared__ uint32_t ids[kShapeCells];
  __shared__ unsigned long long rank_masks[kMaxRanks][4];
  __shared__ uint8_t order[kMaxCombo], packs[kMaxCombo];          // level assignments rank by rank; their levels, in table order
  const DevParams* __restrict__ P = A.P;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t nranks = A.nranks, npass = A.npass, nops = A.nops, NL = A.NL, G = A.G, log2V = A.log2V, V = 1u << log2V, ndt = A.ndt, nwp = A.nwp, nw = nwp << ndt;
  const uint32_t lg_shapes = kLgShapeCells - lg_cells, s0 = blockIdx.x << lg_shapes;          // the workgroup's first shape of the level
  const ShapeRec* __restrict__ recs = all_recs + first + s0;
  const uint32_t info = P->combo_info[tid];
  const uint32_t my_coef = reinterpret_cast<const uint32_t*>(P->mcoef)[tid & 127u];
  // which of the wave's cells fit
  uint32_t here = 0;
#pragma unroll
  for (uint32_t j = 0; j < 4; j++) {
    const uint32_t x = wave * 256u + j * 64u, slot = x >> lg_cells, cell = (x & ((1u << lg_cells) - 1u)) + lane;
    if (s0 + slot < n_shapes && cell < G) {
      const uint32_t c = cell >> log2V, combo = c / npass, pass = c - combo * npass, dt = cell & ((1u << ndt) - 1u);
      here |= (uint32_t)(masks[((size_t)recs[slot].shape * npass + pass) * nw + dt * nwp + (combo >> 6)] >> (combo & 63u) & 1ull) << j;
    }
  }
  {
    const uint32_t pack = info & 0xFFu, rank = tid < P->ncombo ? (uint32_t)__popc(pack & 0x55u) + 2u * (uint32_t)__popc(pack & 0xAAu) : ~0u;
    uint32_t at = 0;
    for (uint32_t r = 0; r < nranks; r++) {
      const unsigned long long m = __ballot(rank == r);
      if (lane == 0) rank_masks[r][wave] = m;
      at = rank == r ? ranks.at[r] + (uint32_t)__popcll(m & ((1ull << lane) - 1ull)) : at;
    }
    packs[tid] = (uint8_t)pack;
    if (tid < 128) coef[tid] = my_coef;
    __syncthreads();
    if (rank != ~0u) {
      for (uint32_t w = 0; w < wave; w++) at += (uint32_t)__popcll(rank_masks[rank][w]);
      order[at] = (uint8_t)tid;
    }
  }
  for (uint32_t i = tid; i < (64u * kChanges) << lg_shapes; i += 256u) {
    const uint32_t row = i >> 2, dst = i & 3u, xx = LAY ? row & 1u : 0u, src = row / kChanges & 3u, op = row / kChanges >> 2 & 3u, slot = row / kChanges >> 4;
    const uint32_t k = coef[((op * 4u + src) * 4u + dst) * 2u + xx];
    uint64_t p = k;
    if (dst < 3) {
      const uint64_t numel = s0 + slot < n_shapes ? recs[slot].numel[op] : 0;
      p = !k ? 1ull << 63 : SMALL ? (uint64_t)k * (uint32_t)numel : mul_or_limit(k, numel);
    }
    prices[row][dst] = p;
  }
  uint32_t n_rw = 0, ovf = 0, over = 0, over2 = 0;
  // ---- tiles, microkernels, bufferize: a lane per cell, 64 cells of one shape at a time
#pragma unroll 1
  for (uint32_t j = 0; j < 4; j++) {
    const uint32_t x = wave * 256u + j * 64u, slot = x >> lg_cells, cell = (x & ((1u << lg_cells) - 1u)) + lane;
    Best e{kInf, kNotHere | kNone};
    if ((here >> j) & 1u) {
      const ShapeRec& R = recs[slot];
      const uint32_t cnts = R.tile_cnt, mk_var = R.mk_var, at = R.shape * G + cell;
      e.id = kNone;
      // the lists of the dimensions one after the other, those of the parallel loops (b, m, n) behind them
      const uint32_t c0 = MN ? 0u : cnts & 0xFFu, c1 = (cnts >> 8) & 0xFFu, c2 = MN ? 0u : (cnts >> 16) & 0xFFu, c3 = cnts >> 24;
      const uint32_t b1 = c0, b2 = c0 + c1, b3 = b2 + c2, n_serial = b3 + c3, n_all = PAR ? n_serial + b2 + c3 : n_serial;
      const uint32_t o0 = R.tile_lo[0], o1 = R.tile_lo[1] - b1, o2 = R.tile_lo[2] - b2, o3 = R.tile_lo[3] - b3;
      for (uint32_t t0 = 0; t0 < n_all; t0 += kShapeBatch) {
        TileStep st[kShapeBatch];
        uint64_t sub[kShapeBatch];
#pragma unroll
        for (uint32_t u = 0; u < kShapeBatch; u++) {
          uint32_t t = t0 + u < n_all ? t0 + u : n_all - 1u;
          const bool loop = PAR && t >= n_serial;
          if (loop) t -= n_serial;
          uint32_t o = o3;
          if (!MN) { o = t < b3 ? o2 : o; o = t < b2 ? o1 : o; o = t < b1 ? o0 : o; }
          else o = t < b3 ? o1 : o;
          if (loop) { o = o3 + c2; o = t < b2 ? o1 : o; o = t < b1 ? o0 : o; }
          st[u] = steps[o + t];
        }
#pragma unroll
        for (uint32_t u = 0; u < kShapeBatch; u++) {
          const uint64_t* table = A.cost;
          if (PAR && t0 + u >= n_serial) table = A.costM;
          sub[u] = at_cell<SMALL>(table, at - st[u].delta);
        }
#pragma unroll
        for (uint32_t u = 0; u < kShapeBatch; u++) {
          const bool loop = PAR && t0 + u >= n_serial, fin = t0 + u < n_all && (uint32_t)(sub[u] >> 32) != ~0u;
          const uint32_t a = fin ? (loop ? st[u].rounds : st[u].trips) : 0u;
          const uint64_t lo64 = (uint64_t)a * (uint32_t)sub[u] + (loop ? A.sync : A.s);     // (32 x 32 bits + 32 bits: no wrap)
          const uint64_t hi = (uint64_t)a * (uint32_t)(sub[u] >> 32) + (lo64 >> 32);        // bits 32.. of the sum
          over |= (uint32_t)hi;
          over2 |= (uint32_t)(hi >> 32);
          e.take((hi << 32) | (uint32_t)lo64, st[u].id + (loop ? A.par_shift : 0u), fin);
        }
      }
      n_rw += R.n_tile;
      if ((mk_var & 0xFFu) | (MN ? A.has_buf : 0u)) {
        const uint32_t v = cell & (V - 1u), c = cell >> log2V, combo = c / npass, pass = c - combo * npass, pack = packs[combo];
        Eval f;
        f.best = e.cost; f.arg = e.id; f.ovf = 0;
        if (mk_var & 0xFFu) {
          for (uint32_t mm = A.mk_entry[(pack << log2V) + v] & mk_var & 0xFFu; mm; mm &= mm - 1) {
            const uint32_t m = (uint32_t)__ffs((int)mm) - 1u;
            Shape H;
#pragma unroll
            for (int d = 0; d < 4; d++) H.d[d] = P->sizes[d][(R.si >> (8 * d)) & 0xFFu];
            const uint64_t ck = mul_or_limit(P->mk_cost[m], mk_shape_reps(P, H, m));
            if (ck >= kLimit) f.ovf = 1; else consider(f, ck, m);
            n_rw++;
          }
        }
        if (MN && A.has_buf) {
          const uint64_t numel[5] = {R.numel[0], R.numel[1], R.numel[2], R.numel[3], R.numel[4]};
          n_rw += task_bufferize(A, R.si, numel, pack, pass, v, f);
        }
        e.cost = f.best; e.id = f.arg;
        ovf |= f.ovf;
      }
    }
    costs[x + lane] = e.cost;
    ids[x + lane] = e.id;
  }
  __syncthreads();
  // ---- Moves, rank by rank: a few lanes of a wave per item (shape and level of the intermediate), which read and write its cells only
  const uint32_t lg_items = 6u - lg_lanes, items = npass << lg_shapes, per_wave = (items + 3u) / 4u, end = (wave + 1u) * per_wave < items ? (wave + 1u) * per_wave : items;
  for (uint32_t i0 = wave * per_wave; i0 < end; i0 += 1u << lg_items) {
    const uint32_t i = i0 + (lane >> lg_lanes), slot = i / npass, pass = i - slot * npass;
    const bool have = i < end && s0 + slot < n_shapes;
    for (uint32_t r = 1; r < nranks; r++) {
      const uint32_t off = ranks.at[r], n = (ranks.at[r + 1] - off) << log2V;
      for (uint32_t e0 = lane & ((1u << lg_lanes) - 1u); __any(e0 < n); e0 += 1u << lg_lanes) {
        if (have && e0 < n) {
          const uint32_t combo = order[off + (e0 >> log2V)], v = e0 & (V - 1u), pack = packs[combo];
          const uint32_t x = (slot << lg_cells) + (((combo * npass + pass) << log2V) | v);
          const uint32_t tile_id = ids[x];
          if (tile_id < kNotHere) {
            Best e{kNoCost, kNone};
            int32_t high = 0;
#pragma unroll
            for (uint32_t op = 0; op < 4; op++) {
              if (op >= nops) break;
              const uint32_t src = (pack >> A.pack_shift[op]) & 3u, to = x - __umul24(src, A.mstride[op]), lay = LAY ? A.lay_xor[op] : 0u;
              const uint64_t* price = prices[((slot * 4u + op) * 4u + src) * kChanges];
              // what is not finite reads as 2^63 - 1, a Move that does not exist costs 2^63: with either bit 63 is set, or the cost is kNoCost and more
              const auto add = [&](uint64_t t, uint64_t p, uint32_t id) {
                const uint64_t cand = (t & kNoCost) + p;
                high = (int32_t)(cand >> 32) > high ? (int32_t)(cand >> 32) : high;
                e.take(cand, id, true);
              };
#pragma unroll
              for (uint32_t dst = 0; dst < 3; dst++) {
                if (dst >= NL - 1u) break;
                const uint32_t from = to + dst * A.mstride[op], id = A.move_base + op * (NL - 1u) * 4u + dst * 4u;
                add(costs[from], price[dst], id);
                if (lay) add(costs[from ^ lay], price[4 + dst], id + 2u);
              }
              n_rw += (uint32_t)price[3];
            }
            over |= high >= 1 << 30 ? 1u << 30 : 0u;
            Eval f;
            f.best = costs[x]; f.arg = tile_id; f.ovf = 0;
            consider(f, e.cost, e.id, e.id != kNone);
            if (ndt) {
              // to the type without the dtype bit; what does not fit there is (INF, NONE)
#pragma unroll
              for (uint32_t op = 0; op < 2; op++) {
                const uint32_t src = (pack >> A.pack_shift[op]) & 3u, cv_bit = A.cv_bit[op];
                if (!(v & cv_bit)) continue;
                n_rw += (uint32_t)prices[((slot * 4u + op) * 4u + src) * kChanges][3];
                for (uint32_t dst = 0; dst < src; dst++)
                  for (uint32_t xx = 0; xx < (LAY && A.lay_xor[op] ? 2u : 1u); xx++) {
                    const uint64_t t = costs[((x - __umul24(src - dst, A.mstride[op])) ^ (xx ? A.lay_xor[op] : 0u)) & ~cv_bit];
                    const uint32_t k = coef[((op * 4u + src) * 4u + dst) * 2u + xx];
                    const uint64_t numel = recs[slot].numel[op];
                    const bool fin = (uint32_t)(t >> 32) != ~0u && k != 0;
                    const uint64_t cand = t + (SMALL ? (uint64_t)(k + A.convert) * (uint32_t)numel : mul_or_limit((uint64_t)k + A.convert, numel));     // each at most 2^62 when finite: no wrap
                    over |= fin ? (uint32_t)(cand >> 32) : 0u;
                    consider(f, cand, A.move_base + op * (NL - 1u) * 4u + dst * 4u + xx * 2u + 1u, fin);
                  }
              }
            }
            costs[x] = f.best;
            ids[x] = f.arg;
          }
        }
      }
      // (the next rank reads what other lanes of this wave wrote: a wave's LDS operations are done in their order)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  if (lg_cells > 8) __syncthreads();        // (else a wave has taken the items of its own cells)
  // ---- whole lines to the table
#pragma unroll
  for (uint32_t j = 0; j < 4; j++) {
    const uint32_t x = wave * 256u + j * 64u, slot = x >> lg_cells, cell = (x & ((1u << lg_cells) - 1u)) + lane;
    if (s0 + slot < n_shapes && cell < G) {
      const size_t at = (size_t)recs[slot].shape * G + cell;
      A.cost[at] = costs[x + lane];
      A.arg[at] = (uint16_t)ids[x + lane];
    }
  }
  ovf |= (over >> 30) | over2;
  flush_counters(A.ctr, n_rw, ovf);
}

// What an alloc-binding costs beside its body (Section 2, Memory Movement; Section 3): m(src) +
// m(dest) in cache lines, the load Move Spec and, for the accumulated output, the store Move Spec,
// both of fresh tensors.  It depends on the operand's size, the two levels, the two layouts and the
// data types only, so it is tabulated once per table instead of being gathered for every Spec.
// [read only, accumulated][rows][columns][data types][level pair][layout before][layout after];
// kInf: no such Move; kLimit: the sum reaches 2^62.
__device__ __forceinline__ uint64_t add_or_limit(uint64_t a, uint64_t b) {
  return (a >= kLimit || b >= kLimit || a + b >= kLimit) ? kLimit : a + b;
}

__global__ __launch_bounds__(256) void bind_kernel(const DevParams* __restrict__ P, uint64_t* __restrict__ bind, uint32_t n) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  const uint32_t yb = P->yb, NL = P->NL;
  uint32_t r = i;
  const uint32_t y1 = r & ((1u << yb) - 1u); r >>= yb;
  const uint32_t y0 = r & ((1u << yb) - 1u); r >>= yb;
  const uint32_t pr = r % 6u; r /= 6u;
  const uint32_t dc = r % P->bind_d; r /= P->bind_d;
  const uint32_t ci = r % P->nszV; r /= P->nszV;
  const uint32_t ri = r % P->nszV, rmw = r / P->nszV;
  const uint32_t src = pr < 1 ? 1u : pr < 3 ? 2u : 3u, dst = pr - src * (src - 1u) / 2u;
  uint64_t out = kInf;
  if (src < NL && (y0 < 2 || P->xw == 4) && (y1 < 2 || P->xw == 4)) {
    const uint32_t bf = dc ? 1u : 0u, child_bf = dc == 1 ? 1u : 0u;
    const uint64_t numel = (uint64_t)P->sizes[1][ri] * P->sizes[3][ci], line = P->line_bytes;
    const uint64_t lines_s = (numel * (bf ? 2u : 4u) + line - 1) / line, lines_d = (numel * (child_bf ? 2u : 4u) + line - 1) / line;
    const uint64_t groupV = (uint64_t)(ri * P->nszV + ci) * P->GV;
    // both tensors fresh: every physical dimension adjacent, aligned
    const uint32_t top0 = y0 >= 2 ? 3u : 2u, top1 = y1 >= 2 ? 3u : 2u;
    const uint32_t q_load = top0 * P->limV_stride[0] + P->limV_stride[1] + top1 * P->limV_stride[2] + P->limV_stride[3];
    const uint32_t q_store = top1 * P->limV_stride[0] + P->limV_stride[1] + top0 * P->limV_stride[2] + P->limV_stride[3];
    auto variant = [&](uint32_t ys, uint32_t yd, uint32_t fs, uint32_t fd) {
      return (P->layV[0] != kNoBit ? ys << P->layV[0] : 0u) + (P->layV[1] != kNoBit ? yd << P->layV[1] : 0u) +
             (P->dtV[0] != kNoBit ? fs << P->dtV[0] : 0u) + (P->dtV[1] != kNoBit ? fd << P->dtV[1] : 0u);
    };
    const uint64_t c_load = P->costM[groupV + ((src * NL + dst) * P->QV + q_load) * P->VV + variant(y0, y1, bf, child_bf)];
    const uint64_t c_store = rmw ? P->costM[groupV + ((dst * NL + src) * P->QV + q_store) * P->VV + variant(y1, y0, child_bf, bf)] : 0;
    if (c_load != kInf && c_store != kInf) {
      out = add_or_limit(mul_or_limit(lines_s, P->weight[src]), mul_or_limit(lines_d, P->weight[dst]));
      out = add_or_limit(add_or_limit(out, c_load), c_store);
    }
  }
  bind[i] = out;
}

// (INF, NONE) are all-ones bytes: stream 16 bytes per lane and store over both tables.
__global__ __launch_bounds__(256) void fill_ones_kernel(uint4* __restrict__ p, size_t n16) {
  const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u);
  for (size_t i = (size_t)blockIdx.x * 256u + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256u) p[i] = ones;
}

// The same in workgroups that end after 16 KB each: beside the latency-bound kernels of another
// stream the compute units' wave slots then turn over all the time, and those kernels' workgroups
// are placed as soon as they are launched (a grid of workgroups that live as long as the whole
// stream of stores holds every slot until it ends).
// Two stretches in one launch.
__global__ __launch_bounds__(256) void fill_ones_short_kernel(uint4* __restrict__ p, size_t n16, uint32_t blocks, uint4* __restrict__ q, size_t m16) {
  const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u);
  const bool second = blockIdx.x >= blocks;
  uint4* to = second ? q : p;
  const size_t n = second ? m16 : n16, i0 = (size_t)(second ? blockIdx.x - blocks : blockIdx.x) * 1024u + threadIdx.x;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const size_t i = i0 + (size_t)k * 256u;
    if (i < n) to[i] = ones;
  }
}

void launch_fill_ones(void* p, size_t bytes, hipStream_t stream) {
  const size_t n16 = bytes / 16;
  if (n16) {
    const size_t blocks = (n16 + 255) / 256;
    hipLaunchKernelGGL(fill_ones_kernel, dim3((uint32_t)(blocks < 16384 ? blocks : 16384)), dim3(256), 0, stream,
                       (uint4*)p, n16);
  }
  if (bytes % 16) (void)hipMemsetAsync((char*)p + n16 * 16, 0xFF, bytes % 16, stream);
}

// A table: (INF, NONE) everywhere.  (fewer than 2^32 Specs: the grid stays below 2^22 workgroups)
void launch_prefill(uint64_t* cost, uint16_t* arg, size_t n, hipStream_t stream) {
  const size_t n16 = n / 2, m16 = n / 8;
  const uint32_t blocks = (uint32_t)((n16 + 1023) / 1024), more = (uint32_t)((m16 + 1023) / 1024);
  if (blocks + more) hipLaunchKernelGGL(fill_ones_short_kernel, dim3(blocks + more), dim3(256), 0, stream, (uint4*)cost, n16, blocks, (uint4*)arg, m16);
  if (n % 2) (void)hipMemsetAsync(cost + n16 * 2, 0xFF, 8, stream);
  if (n % 8) (void)hipMemsetAsync(arg + m16 * 8, 0xFF, n % 8 * 2, stream);
}

// ---------------------------------------------------------------- memory bounds as coordinates
// Sections 2.2 and 2.4.4: a Spec carries, per level of finite capacity, the bytes an implementation
// may still allocate there; a Move allocates the moved operand's buffer in its destination, so it
// needs that many bytes of the destination's bound and leaves its body the rest, rounded down to
// a power of two (or zero).  There is no admissibility test: the bounds decide.
//
// A Move lowers the sum of the operand levels (the rank) within a shape, and a tile goes to the
// same level assignment of a smaller shape (a lower dependency level of shapes), so the Specs of
// (level l, rank r) depend only on (l, r' < r) and (l' < l, r): all pairs on one diagonal
// l + r = d are independent, and one launch takes a whole diagonal, one segment of workgroups per
// pair.  Every candidate is a gather from finished entries.  Specs are numbered (shape of the
// level, level assignment of the rank, level of the fused Spec's intermediate, bound vector,
// variant), variant fastest.  A bufferize (fused Spec) allocates the intermediate in its level:
// it needs 4 * m * n bytes of that level's bound, and both stages get the rest, rounded down.
//
// Move Specs (Section 2.2; kind kKindV) are also gathers from finished entries: two tensors, no
// Move rewrites; where a bounded lattice has its bounds they have the abstract values of Section
// 2.4.3 (contiguousness and aligned flag of source and destination), which a tile changes and the
// vector-move microkernels test.
// ---- a wave per stretch of one (shape, level assignment)
// What the candidates of a Spec are (which Moves and tiles exist, their constants, the groups their
// sub-Specs lie in, the bytes a Move allocates) depends on the shape and the level assignment only;
// the bound vector (or abstract vector) and the variant pick the entry inside those groups.  So a
// wave stays on one such unit of Q * V consecutive entries: its lanes first work out one candidate
// each (UnitMove, UnitTile), then every lane walks the candidates, whose constants it gets as
// scalars (readlane), and its own share of one is an offset, a read and a comparison.  The
// candidates come in the order of their ids, so a strictly lower cost is all that has to be tested.
// With a lane per Spec that decoded its own shape and levels the kernel was bound by those
// instructions (config 7, 41 M Specs, 413 M candidates: fill 1.84 ms, now 1.00 ms, about half of
// it instruction issue; config 12's Move table, 16.8 M Specs: 0.84 ms, now 0.42 ms).
// Needs enough entries per unit to fill a wave (kUnitLanes); narrower units stay with the kernel below.
constexpr uint32_t kUnitLanes = 32;
constexpr int kUnitBatch = 8;         // candidates whose reads are in flight together

// A buffer of `bytes` out of a bound q (q = 0: nothing, else 2^(q-1) bytes): the least q that holds
// it, and how far that q falls when the rest is rounded down to a power of two.  Any larger q falls
// by one: 2^(q-1) - bytes is then at least half of 2^(q-1), but less than it.
struct BoundStep { uint32_t qmin, dmin; };
__device__ __forceinline__ BoundStep bound_step(uint64_t bytes) {
  const uint32_t lg = bytes <= 1 ? 0u : 64u - (uint32_t)__clzll((long long)(bytes - 1));
  const uint64_t left = (1ull << lg) - bytes;
  BoundStep b;
  b.qmin = lg + 1;
  b.dmin = b.qmin - (left ? 64u - (uint32_t)__clzll((long long)left) : 0u);
  return b;
}

// Section 2.4.3 for one tile of a shape, for every layout at once: 4 bits per layout y at 4 * y,
// bits 0..1 = the most contiguousness that is left, bits 2 and 3 = the tile's suffix products are
// whole cache lines for 4- and for 2-byte elements (tile_abstract's `keep` and `lines_ok`).
__device__ __forceinline__ uint32_t tile_word(const DevParams* __restrict__ P, uint32_t rows, uint32_t cols, uint32_t r2, uint32_t c2) {
  const uint32_t strip = P->strip ? P->strip : 1u;
  uint32_t word = 0;
  for (uint32_t y = 0; y < P->xw; y++)
#pragma unroll
    for (uint32_t bf = 0; bf < 2; bf++) {
      uint32_t keep, line_ok;
      // (a tensor that is aligned and contiguous in all its dimensions keeps what the tile allows)
      tile_abstract(y, rows, cols, r2, c2, bf ? 2u : 4u, strip, P->line_bytes, P->line_mask, y >= 2 ? 3u : 2u, 1u, keep, line_ok);
      word |= keep << (4 * y) | line_ok << (4 * y + 2 + bf);
    }
  return word;
}

// One lane's candidate of the unit.
struct UnitTile {
  uint32_t cell, trips, id, word;      // first entry of the child's unit; trip count; rewrite id; Move Specs: tile_word
};
struct UnitMove {
  bool exists;
  uint32_t delta;                      // the body's unit lies this many entries before this one
  uint32_t id, b_lo, b_hi;             // coefficient * elements, at most kLimit
  uint32_t steps;                      // bound_step's qmin of the buffer at 4 (byte 0) and at 2 bytes per element (byte 1); byte 2: bit of the bound in qdec
  uint32_t stride, fall4, fall2;       // stride of the destination's bound; dmin * stride at 4 and at 2 bytes (all 0, and qmin 0, if unbounded)
  uint32_t vxor, vclear, need;         // variant of the body = (variant ^ vxor) & ~vclear; lanes with the bit `need` only (0: all)
  uint32_t half;                       // variant bit that says the moved operand has 2 bytes per element (0: never, ~0: always)
};

// MODE 0: memory bounds as coordinates; 1: Move Specs (no Moves: all level assignments of a
// dependency level of shapes in one launch, and the segments' rank is not used).  R: entries per
// lane and step; two share a candidate's constants where a wave has that many (config 7's fill 1.24 ms
// with one, 1.19 ms with two).
template <int MODE, int R>
__global__ __launch_bounds__(256) void fill_units_kernel(const DevParams* __restrict__ P,
                                                         const uint32_t* __restrict__ all_level_shapes, const BoundSegs segs,
                                                         uint64_t* cost, uint16_t* __restrict__ arg,
                                                         Counters* __restrict__ ctr) {
  __shared__ uint32_t wave_n[4], wave_adm[4];
  uint32_t seg = 0;
  while (seg + 1 < segs.n && blockIdx.x >= segs.block0[seg + 1]) seg++;
  const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t log2V = P->log2V, V = 1u << log2V, Q = P->Q, npass = P->npass, nops = P->nops, QV = Q << log2V;
  const uint32_t c0 = MODE == 1 ? 0u : P->rank_off[segs.rank[seg]], ncr = MODE == 1 ? P->ncombo : P->rank_off[segs.rank[seg] + 1] - c0;
  const uint32_t wv = (blockIdx.x - segs.block0[seg]) * 4u + wave;
  const uint32_t unit = wv / segs.waves_per_unit, chunk = wv - unit * segs.waves_per_unit;
  uint32_t n_rw = 0, n_adm = 0, ovf = 0;
  if (unit < segs.n_shapes[seg] * ncr * npass) {
    const uint32_t sl = unit / (ncr * npass), rem = unit - sl * ncr * npass;
    const uint32_t ci = rem / npass, pass = rem - ci * npass;
    const uint32_t shape = all_level_shapes[segs.first_shape[seg] + sl];
    Shape S;
    load_shape(P, shape, S);
    const uint32_t pack = P->combo_info[c0 + ci] & 0xFFu;
    uint32_t combo = 0, lv[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; i++)
      if ((uint32_t)i < nops) { lv[i] = (pack >> P->pack_shift[i]) & 3u; combo += lv[i] * P->lvpow[i]; }
    const uint32_t row = (combo * npass + pass) * QV;          // the unit's first entry inside the group
    const uint32_t first_cell = shape * P->G + row;            // (cells of a table fit 32 bits)
    uint64_t* mine = cost + first_cell;

    // microkernels whose shape predicate holds
    uint32_t mk_shape = 0;
    for (uint32_t j = 0; j < P->nmk; j++) mk_shape |= (mk_shape_reps(P, S, j) ? 1u : 0u) << j;

    // the unit's Moves, lane t = ((operand * 3 + destination) * 2 + transposed) * 2 + converted (at most 48)
    UnitMove mv;
    mv.exists = false; mv.delta = mv.id = mv.b_lo = mv.b_hi = mv.steps = mv.stride = mv.fall4 = mv.fall2 = mv.vxor = mv.vclear = mv.need = mv.half = 0;
    bool halves = false;       // some Move's operand may have 2 bytes per element
    if (MODE == 0) {
      const uint32_t i = lane / 12u, dst = lane / 4u - 3u * i, xx = (lane >> 1) & 1u, cv = lane & 1u;
      if (i < nops) {
        const uint32_t src = i == 0 ? lv[0] : i == 1 ? lv[1] : i == 2 ? lv[2] : lv[3];
        const bool has_dt = P->dt_bit[i] != kNoBit, has_lay = P->lay_bit[i] != kNoBit;
        const uint32_t coef = dst < src && (!xx || has_lay) && (!cv || (P->can_convert[i] && has_dt)) ? P->mcoef[i][src][dst][xx] : 0u;
        if (coef) {
          const uint64_t numel = i == 0 ? S.numel[0] : i == 1 ? S.numel[1] : i == 2 ? S.numel[2] : S.numel[3];
          const uint64_t bc = mul_or_limit((uint64_t)coef + (cv ? P->convert : 0u), numel);
          const uint32_t dtbit = has_dt ? 1u << P->dt_bit[i] : 0u, la = P->lim_of_level[dst];
          mv.exists = true;
          mv.delta = (src - dst) * P->lvpow[i] * npass * QV;
          mv.id = P->move_base + ((i * (P->NL - 1u) + dst) * 2u + xx) * 2u + cv;
          mv.b_lo = (uint32_t)bc; mv.b_hi = (uint32_t)(bc >> 32);
          if (la != kNoBit) {
            const BoundStep s4 = bound_step(numel * 4u), s2 = bound_step(numel * 2u);
            mv.steps = s4.qmin | s2.qmin << 8 | (8u * la) << 16;
            mv.stride = P->lim_stride[la]; mv.fall4 = s4.dmin * mv.stride; mv.fall2 = s2.dmin * mv.stride;
          }
          mv.vxor = xx ? 1u << P->lay_bit[i] : 0u;
          mv.vclear = cv ? dtbit : 0u;
          mv.need = cv ? dtbit : 0u;
          mv.half = cv ? 0u : has_dt ? dtbit : P->base_bf16[i] ? ~0u : 0u;     // element size after the Move
        }
      }
      halves = __any(mv.half != 0);
    }
    const unsigned long long moves = __ballot(mv.exists);
    const bool variants = log2V != 0;

    // its tiles, one per lane; where there are more than 64, the further ones in rounds
    uint32_t n_tile = 0;
#pragma unroll
    for (int d = 0; d < 4; d++) n_tile += P->tile_dim_ok[d] ? P->tile_off[d][S.si[d] + 1] - P->tile_off[d][S.si[d]] : 0u;
    UnitTile tl;
    tl.cell = tl.trips = tl.id = tl.word = 0;
    auto fetch_tiles = [&](uint32_t t0) {
      if (t0 + lane < n_tile) {
        uint32_t first = 0, td = 0, at = 0;
#pragma unroll
        for (int d = 0; d < 4; d++) {
          const uint32_t lo = P->tile_off[d][S.si[d]];
          const uint32_t cnt = P->tile_dim_ok[d] ? P->tile_off[d][S.si[d] + 1] - lo : 0u;
          if (t0 + lane >= first && t0 + lane < first + cnt) { td = d; at = lo + (t0 + lane - first); }
          first += cnt;
        }
        const TileEntry te = P->tiles[at];
        const uint32_t sj = td == 0 ? S.si[0] : td == 1 ? S.si[1] : td == 2 ? S.si[2] : S.si[3];
        tl.cell = (shape - (sj - te.jt) * P->shape_stride[td]) * P->G + row;
        tl.trips = te.trips;
        tl.id = P->tile_base + td * P->maxs + te.jt;
        if (MODE == 1)
          tl.word = tile_word(P, (uint32_t)S.d[1], (uint32_t)S.d[3], td == 1 ? P->sizes[1][te.jt] : (uint32_t)S.d[1],
                              td == 3 ? P->sizes[3][te.jt] : (uint32_t)S.d[3]);
      }
    };
    fetch_tiles(0);

    const uint32_t x_end = QV < (chunk + 1) * segs.lanes_per_wave ? QV : (chunk + 1) * segs.lanes_per_wave;
    for (uint32_t x0 = chunk * segs.lanes_per_wave; x0 < x_end; x0 += 64 * R) {
      uint32_t x[R], q[R], v[R], qd[R], best_id[R], over = 0;    // over: OR of the high words of all finite candidates
      uint64_t best[R];
      bool on[R], live[R];
      uint32_t y[R][2], bfl[R][2];
#pragma unroll
      for (int r = 0; r < R; r++) {
        on[r] = x0 + 64 * r + lane < x_end;
        x[r] = on[r] ? x0 + 64 * r + lane : x_end - 1;
        q[r] = x[r] >> log2V; v[r] = x[r] & (V - 1u);
        qd[r] = P->qdec[q[r]];                                   // the bound vector's (abstract vector's) axes, a byte each
        best[r] = kInf; best_id[r] = kNone;
        live[r] = on[r];
        if (MODE == 1) {
#pragma unroll
          for (int ts = 0; ts < 2; ts++) {
            y[r][ts] = P->lay_bit[ts] != kNoBit ? (v[r] >> P->lay_bit[ts]) & ((1u << P->lay_w[ts]) - 1u) : 0u;
            bfl[r][ts] = P->dt_bit[ts] != kNoBit ? (v[r] >> P->dt_bit[ts]) & 1u : P->base_bf16[ts];
            // no such tensor: a packed layout with a broken strip, more adjacent dimensions than the tensor can have
            if (P->xw == 4)
              live[r] = live[r] && layout_fits(y[r][ts], (uint32_t)S.d[3], P->strip) &&
                        ((qd[r] >> (16 * ts)) & 0xFFu) <= max_contig(y[r][ts], (uint32_t)S.d[3], P->strip);
          }
          n_adm += (uint32_t)__popcll(__ballot(live[r]));
        }
      }

      for (uint32_t left = mk_shape; left; left &= left - 1) {
        const uint32_t j = (uint32_t)__ffs((int)left) - 1u;
        const uint64_t k = mul_or_limit(P->mk_cost[j], mk_shape_reps(P, S, j));
#pragma unroll
        for (int r = 0; r < R; r++) {
          bool ok = live[r] && ((P->mk_entry[(pack << log2V) + v[r]] >> j) & 1u);
          if (MODE == 1 && P->mk_kind[j] >= 6u) {
            // vector moves: the inner dimension of both tensors adjacent in memory; the aligned form: both aligned;
            // a row of whole strips: the strips must be whole vectors
            ok = ok && (qd[r] & 0xFFu) >= 1u && ((qd[r] >> 16) & 0xFFu) >= 1u;
            if (P->mk_kind[j] == 7u) ok = ok && ((qd[r] >> 8) & 1u) && ((qd[r] >> 24) & 1u);
            if (P->xw == 4 && S.d[3] >= P->strip && P->strip % P->mk_lanes[j] != 0) ok = ok && y[r][0] < 2 && y[r][1] < 2;
          }
          over |= ok ? (uint32_t)(k >> 32) : 0u;
          const bool better = ok && k < best[r];
          best[r] = better ? k : best[r];
          best_id[r] = better ? j : best_id[r];
          n_rw += (uint32_t)__popcll(__ballot(ok));
        }
      }

      if (MODE == 0) {
        for (unsigned long long todo = moves; todo;) {
          uint64_t sub[kUnitBatch][R];
          bool ok[kUnitBatch][R];
          unsigned long long left = todo;
#pragma unroll
          for (int u = 0; u < kUnitBatch; u++) {
#pragma unroll
            for (int r = 0; r < R; r++) { ok[u][r] = false; sub[u][r] = kInf; }
            if (left) {
              const uint32_t t = (uint32_t)__builtin_ctzll(left);
              left &= left - 1;
              const uint32_t steps = lane_of(mv.steps, t), stride = lane_of(mv.stride, t), fall4 = lane_of(mv.fall4, t);
              const char* to = (const char*)(mine - lane_of(mv.delta, t));
#pragma unroll
              for (int r = 0; r < R; r++) {
                uint32_t qmin = steps & 0xFFu, fall = fall4;
                if (halves) {
                  const uint32_t half = lane_of(mv.half, t), fall2 = lane_of(mv.fall2, t);
                  const bool h = (v[r] & half) != 0 || half == ~0u;
                  qmin = h ? (steps >> 8) & 0xFFu : qmin;
                  fall = h ? fall2 : fall;
                }
                const uint32_t qa = (qd[r] >> (steps >> 16)) & 0xFFu;
                ok[u][r] = live[r] && qa >= qmin;
                uint32_t at = q[r] - (qa > qmin ? stride : fall);
                if (variants) {
                  const uint32_t need = lane_of(mv.need, t);
                  ok[u][r] = ok[u][r] && (v[r] & need) == need;
                  at = (at << log2V) + ((v[r] ^ lane_of(mv.vxor, t)) & ~lane_of(mv.vclear, t));
                }
                at = ok[u][r] ? at << 3 : 0u;        // the others read any finished entry and drop it
                sub[u][r] = *(const uint64_t*)(to + at);
              }
            }
          }
#pragma unroll
          for (int u = 0; u < kUnitBatch; u++) {
            if (todo) {
              const uint32_t t = (uint32_t)__builtin_ctzll(todo);
              todo &= todo - 1;
              const uint64_t b = (uint64_t)lane_of(mv.b_hi, t) << 32 | lane_of(mv.b_lo, t);
              const uint32_t id = lane_of(mv.id, t);
#pragma unroll
              for (int r = 0; r < R; r++) {
                const bool fin = ok[u][r] && (uint32_t)(sub[u][r] >> 32) != ~0u;
                const uint64_t cand = sub[u][r] + b;                // each at most 2^62: no wrap
                over |= fin ? (uint32_t)(cand >> 32) : 0u;
                const bool better = fin && cand < best[r];
                best[r] = better ? cand : best[r];
                best_id[r] = better ? id : best_id[r];
                n_rw += (uint32_t)__popcll(__ballot(ok[u][r]));
              }
            }
          }
        }
      }

      // tiles: the same entry of a smaller shape's group (a Move Spec's: the entry with what the tile leaves)
      const uint64_t s_loop = P->s;
      for (uint32_t t0 = 0; t0 < n_tile; t0 += 64) {
        if (n_tile > 64) fetch_tiles(t0);
        const uint32_t n_here = n_tile - t0 < 64u ? n_tile - t0 : 64u;
        for (uint32_t u0 = 0; u0 < n_here; u0 += kUnitBatch) {
          uint64_t sub[kUnitBatch][R];
#pragma unroll
          for (int u = 0; u < kUnitBatch; u++) {
#pragma unroll
            for (int r = 0; r < R; r++) sub[u][r] = kInf;
            if (u0 + u < n_here) {
              const char* to = (const char*)(cost + lane_of(tl.cell, u0 + u));
              const uint32_t word = MODE == 1 ? lane_of(tl.word, u0 + u) : 0u;
#pragma unroll
              for (int r = 0; r < R; r++) {
                uint32_t at = x[r];
                if (MODE == 1) {
                  uint32_t qc = 0;
#pragma unroll
                  for (int ts = 0; ts < 2; ts++) {
                    const uint32_t f = word >> (4 * y[r][ts]), keep = f & 3u, lines = (f >> (2 + bfl[r][ts])) & 1u;
                    const uint32_t contig = (qd[r] >> (16 * ts)) & 0xFFu, aligned = (qd[r] >> (16 * ts + 8)) & 1u;
                    const uint32_t nd = y[r][ts] >= 2 ? 3u : 2u;
                    qc += (contig < keep ? contig : keep) * P->lim_stride[2 * ts] + (contig == nd ? aligned & lines : 0u) * P->lim_stride[2 * ts + 1];
                  }
                  at = (qc << log2V) + v[r];
                }
                sub[u][r] = *(const uint64_t*)(to + (at << 3));
              }
            }
          }
#pragma unroll
          for (int u = 0; u < kUnitBatch; u++) {
            if (u0 + u < n_here) {
              const uint32_t a = lane_of(tl.trips, u0 + u), id = lane_of(tl.id, u0 + u);
#pragma unroll
              for (int r = 0; r < R; r++) {
                const bool fin = live[r] && (uint32_t)(sub[u][r] >> 32) != ~0u;
                const uint64_t lo = (uint64_t)a * (uint32_t)sub[u][r];
                const uint64_t hi = (uint64_t)a * (uint32_t)(sub[u][r] >> 32) + (lo >> 32);     // bits 32.. of the product
                const uint64_t cand = ((hi << 32) | (uint32_t)lo) + s_loop;
                // (the product's own bits count as well: the sum may pass 2^64)
                over |= fin ? (uint32_t)(cand >> 32) | (uint32_t)hi | ((uint32_t)(hi >> 32) ? 1u << 30 : 0u) : 0u;
                const bool better = fin && cand < best[r];
                best[r] = better ? cand : best[r];
                best_id[r] = better ? id : best_id[r];
              }
            }
          }
        }
      }
#pragma unroll
      for (int r = 0; r < R; r++) n_rw += n_tile * (uint32_t)__popcll(__ballot(live[r]));

      // bufferize (fused Spec): the Matmul into the intermediate at level `pass`, then the bias-add + ReLU out of it
      if (MODE == 0 && P->kind == kKindF) {
        const uint32_t la = P->lim_of_level[pass], NL = P->NL;
        const BoundStep step = bound_step(S.numel[4] * 4u);
        const uint32_t zc = pass == 0 ? P->zero[0] : pass == 1 ? P->zero[1] : pass == 2 ? P->zero[2] : P->zero[3];
        const uint64_t z = mul_or_limit(zc, S.numel[4]);
        const uint64_t* __restrict__ at_m = P->costM + (uint64_t)((S.si[1] * P->nkM + S.si[2] + P->kM_first) * P->nsz[3] + S.si[3]) * P->GM +
                                            (uint64_t)((lv[0] * NL + lv[1]) * NL + pass) * Q * P->VM;
        const uint64_t* __restrict__ at_e = P->costE + (uint64_t)(S.si[1] * P->nszE_n + S.si[3]) * P->GE +
                                            (uint64_t)((pass * NL + lv[2]) * NL + lv[3]) * Q * P->VE;
#pragma unroll
        for (int r = 0; r < R; r++) {
          uint32_t qc = q[r];
          bool fits = live[r];
          if (la != kNoBit) {
            const uint32_t qa = (qd[r] >> (8u * la)) & 0xFFu;
            fits = fits && qa >= step.qmin;
            qc = q[r] - (qa > step.qmin ? 1u : step.dmin) * P->lim_stride[la];
          }
          const uint32_t y0 = P->lay_bit[0] != kNoBit ? (v[r] >> P->lay_bit[0]) & 1u : 0u;
          const uint32_t y1 = P->lay_bit[1] != kNoBit ? (v[r] >> P->lay_bit[1]) & 1u : 0u;
          const uint32_t y3 = P->lay_bit[3] != kNoBit ? (v[r] >> P->lay_bit[3]) & 1u : 0u;
          const uint32_t vm = (P->layM[0] != kNoBit ? y0 << P->layM[0] : 0u) + (P->layM[1] != kNoBit ? y1 << P->layM[1] : 0u);
          const uint32_t ve = P->layE[2] != kNoBit ? y3 << P->layE[2] : 0u;
          const uint64_t cm = fits ? at_m[qc * P->VM + vm] : kInf, ce = fits ? at_e[qc * P->VE + ve] : kInf;
          if (cm != kInf && ce != kInf) {
            const uint64_t zm = z + cm, cand = zm + ce;       // each term at most 2^62: no wrap
            over |= (uint32_t)((z | zm | cand) >> 32);
            if (cand < best[r]) { best[r] = cand; best_id[r] = P->buf_id; }
          }
          n_rw += (uint32_t)__popcll(__ballot(fits));
        }
      }

#pragma unroll
      for (int r = 0; r < R; r++)
        if (on[r]) {
          mine[x[r]] = best[r];
          arg[first_cell + x[r]] = (uint16_t)best_id[r];
        }
      ovf |= over >> 30;
    }
  }
  // rewrites evaluated (and Specs that exist): one atomic each per workgroup
  if (lane == 0) { wave_n[wave] = n_rw; wave_adm[wave] = n_adm; }
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t n = wave_n[0] + wave_n[1] + wave_n[2] + wave_n[3];
    if (n) atomicAdd(&ctr->n_rewrites[blockIdx.x % kCtrSlots], (unsigned long long)n);
    const uint32_t na = wave_adm[0] + wave_adm[1] + wave_adm[2] + wave_adm[3];
    if (MODE != 0 && na) atomicAdd(&ctr->n_admissible[blockIdx.x % kCtrSlots], (unsigned long long)na);
  }
  if (ovf) atomicOr(&ctr->overflow, 1u);
}

// A lane per Spec: bounded lattices with fewer than kUnitLanes entries per level assignment.
__global__ __launch_bounds__(256) void fill_bounded_kernel(const DevParams* __restrict__ P,
                                                           const uint32_t* __restrict__ all_level_shapes, const BoundSegs segs,
                                                           uint64_t* cost, uint16_t* __restrict__ arg,
                                                           Counters* __restrict__ ctr) {
  __shared__ uint32_t wave_n[4];
  uint32_t seg = 0;
  while (seg + 1 < segs.n && blockIdx.x >= segs.block0[seg + 1]) seg++;
  const uint32_t rank = segs.rank[seg], n_level_shapes = segs.n_shapes[seg];
  const uint32_t* __restrict__ level_shapes = all_level_shapes + segs.first_shape[seg];
  const uint32_t V = P->V, Q = P->Q, npass = P->npass, nops = P->nops;
  const uint32_t c0 = P->rank_off[rank], ncr = P->rank_off[rank + 1] - c0;
  const uint64_t per_shape = (uint64_t)ncr * npass * Q * V;
  const uint64_t t = (uint64_t)(blockIdx.x - segs.block0[seg]) * 256u + threadIdx.x;
  const bool active = t < per_shape * n_level_shapes;
  Eval e;
  e.best = kInf; e.arg = kNone; e.n = 0; e.ovf = 0;
  if (active) {
    // (an active lane's index is below the number of Specs of the lattice, which fits 32 bits)
    const uint32_t sl = (uint32_t)t / (uint32_t)per_shape;
    uint32_t r = (uint32_t)t - sl * (uint32_t)per_shape;
    const uint32_t ci = r / (npass * Q * V);
    r -= ci * npass * Q * V;
    const uint32_t pass = r / (Q * V);
    r -= pass * Q * V;
    const uint32_t q = r / V, v = r - q * V;
    const uint32_t shape = level_shapes[sl];
    Shape S;
    load_shape(P, shape, S);
    const uint32_t pack = P->combo_info[c0 + ci] & 0xFFu;
    uint32_t lv[4] = {0, 0, 0, 0}, combo = 0;
#pragma unroll
    for (int i = 0; i < 4; i++)
      if ((uint32_t)i < nops) { lv[i] = (pack >> P->pack_shift[i]) & 3u; combo += lv[i] * P->lvpow[i]; }
    uint32_t qi[4] = {0, 0, 0, 0};
    {
      uint32_t rem = q;
#pragma unroll
      for (int a = 0; a < 4; a++)
        if ((uint32_t)a < P->nlim) { qi[a] = rem / P->lim_stride[a]; rem -= qi[a] * P->lim_stride[a]; }
    }
    const uint64_t group = (uint64_t)shape * P->G;
    const uint32_t off = ((combo * npass + pass) * Q + q) * V + v;
    // microkernels
    const uint32_t mm = P->mk_entry[pack * V + v];
    for (uint32_t j = 0; j < P->nmk; j++) {
      if (!((mm >> j) & 1u)) continue;
      const uint64_t reps = mk_shape_reps(P, S, j);
      if (!reps) continue;
      const uint64_t k = mul_or_limit(P->mk_cost[j], reps);
      if (k >= kLimit) e.ovf = 1; else consider(e, k, j);
      e.n++;
    }

    // Moves
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if ((uint32_t)i >= nops) continue;
      const uint32_t src = lv[i];
      const bool has_dt = P->dt_bit[i] != kNoBit, has_lay = P->lay_bit[i] != kNoBit;
      const uint32_t bf = has_dt ? (v >> P->dt_bit[i]) & 1u : P->base_bf16[i];
      const uint64_t numel = S.numel[i];
      for (uint32_t dst = 0; dst < src; dst++)
        for (uint32_t x = 0; x < 2; x++)
          for (uint32_t cv = 0; cv < 2; cv++) {
            if (x && !has_lay) continue;
            if (cv && !(P->can_convert[i] && has_dt && bf)) continue;
            const uint32_t child_bf = cv ? 0u : bf;
            const uint32_t coef = P->mcoef[i][src][dst][x];
            if (!coef) continue;
            uint32_t qc = q;
            const uint32_t la = P->lim_of_level[dst];
            if (la != kNoBit) {
              const uint32_t qa = la == 0 ? qi[0] : la == 1 ? qi[1] : la == 2 ? qi[2] : qi[3];
              const uint64_t bytes = numel * (child_bf ? 2u : 4u);
              const uint64_t have = qa ? 1ull << (qa - 1u) : 0ull;
              if (bytes > have) continue;                       // the buffer does not fit the bound: no such rewrite
              const uint64_t left = have - bytes;
              const uint32_t qn = left ? 64u - (uint32_t)__clzll((long long)left) : 0u;
              qc = q - (qa - qn) * P->lim_stride[la];
            }
            const uint32_t combo_c = combo - (src - dst) * P->lvpow[i];
            uint32_t v_c = v ^ (x ? 1u << P->lay_bit[i] : 0u);
            if (cv) v_c &= ~(1u << P->dt_bit[i]);
            const uint64_t sub = cost[group + (uint64_t)((combo_c * npass + pass) * Q + qc) * V + v_c];
            const uint64_t b = mul_or_limit((uint64_t)coef + (cv ? P->convert : 0u), numel);
            const uint32_t id = P->move_base + (((uint32_t)i * (P->NL - 1u) + dst) * 2u + x) * 2u + cv;
            if (sub != kInf) {
              if (b >= kLimit || sub + b >= kLimit) e.ovf = 1; else consider(e, sub + b, id);
            }
            e.n++;
          }
    }

    // tiles: the same entry of a smaller shape's group
    const uint64_t s = P->s;
#pragma unroll
    for (int d = 0; d < 4; d++) {
      if (!P->tile_dim_ok[d]) continue;
      for (uint32_t te_i = P->tile_off[d][S.si[d]]; te_i < P->tile_off[d][S.si[d] + 1]; te_i++) {
        const TileEntry te = P->tiles[te_i];
        const uint32_t child = shape - (S.si[d] - te.jt) * P->shape_stride[d];
        const uint64_t sub = cost[(uint64_t)child * P->G + off];
        const bool fin = sub != kInf;
        const uint32_t a = te.trips;
        const uint64_t lo = (uint64_t)a * (uint32_t)sub;
        const uint64_t hi = (uint64_t)a * (uint32_t)(sub >> 32) + (lo >> 32);
        const uint64_t c = ((hi << 32) | (uint32_t)lo) + s;
        const bool over = fin & (((hi >> 30) != 0) | (c >= kLimit));
        e.ovf |= over ? 1u : 0u;
        consider(e, c, P->tile_base + (uint32_t)d * P->maxs + te.jt, fin & !over);
        e.n++;
      }
    }
    // bufferize (fused Spec): the Matmul into the intermediate at level `pass`, then the bias-add +
    // ReLU out of it; both read from the bounded tables of those two kinds
    if (P->kind == kKindF) {
      uint32_t qc = q;
      bool fits = true;
      const uint32_t la = P->lim_of_level[pass];
      if (la != kNoBit) {
        const uint32_t qa = la == 0 ? qi[0] : la == 1 ? qi[1] : la == 2 ? qi[2] : qi[3];
        const uint64_t bytes = S.numel[4] * 4u;
        const uint64_t have = qa ? 1ull << (qa - 1u) : 0ull;
        fits = bytes <= have;
        const uint64_t left = fits ? have - bytes : 0ull;
        const uint32_t qn = left ? 64u - (uint32_t)__clzll((long long)left) : 0u;
        qc = fits ? q - (qa - qn) * P->lim_stride[la] : q;
      }
      if (fits) {
        const uint32_t NL = P->NL;
        const uint32_t y0 = P->lay_bit[0] != kNoBit ? (v >> P->lay_bit[0]) & 1u : 0u;
        const uint32_t y1 = P->lay_bit[1] != kNoBit ? (v >> P->lay_bit[1]) & 1u : 0u;
        const uint32_t y3 = P->lay_bit[3] != kNoBit ? (v >> P->lay_bit[3]) & 1u : 0u;
        const uint32_t vm = (P->layM[0] != kNoBit ? y0 << P->layM[0] : 0u) + (P->layM[1] != kNoBit ? y1 << P->layM[1] : 0u);
        const uint32_t ve = P->layE[2] != kNoBit ? y3 << P->layE[2] : 0u;
        const uint32_t xm = (((lv[0] * NL + lv[1]) * NL + pass) * Q + qc) * P->VM + vm;
        const uint32_t xe = (((pass * NL + lv[2]) * NL + lv[3]) * Q + qc) * P->VE + ve;
        const uint64_t cm = P->costM[(uint64_t)((S.si[1] * P->nkM + S.si[2] + P->kM_first) * P->nsz[3] + S.si[3]) * P->GM + xm];
        const uint64_t ce = P->costE[(uint64_t)(S.si[1] * P->nszE_n + S.si[3]) * P->GE + xe];
        const uint32_t zc = pass == 0 ? P->zero[0] : pass == 1 ? P->zero[1] : pass == 2 ? P->zero[2] : P->zero[3];
        if (cm != kInf && ce != kInf) {
          const uint64_t z = mul_or_limit(zc, S.numel[4]);
          const uint64_t sum = z + cm;          // each term <= 2^62: no wrap
          if (z >= kLimit || sum >= kLimit || sum + ce >= kLimit) e.ovf = 1; else consider(e, sum + ce, P->buf_id);
        }
        e.n++;
      }
    }
    cost[group + off] = e.best;
    arg[group + off] = (uint16_t)e.arg;
  }
  // rewrites evaluated: one atomic per workgroup
  uint32_t n_rw = e.n;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    n_rw += __shfl_down(n_rw, d, 64);
  }
  if ((threadIdx.x & 63u) == 0) wave_n[threadIdx.x >> 6] = n_rw;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t n = wave_n[0] + wave_n[1] + wave_n[2] + wave_n[3];
    if (n) atomicAdd(&ctr->n_rewrites[blockIdx.x % kCtrSlots], (unsigned long long)n);
  }
  if (e.ovf) atomicOr(&ctr->overflow, e.ovf);
}

// One launch over segs: one diagonal (or a part of it), or for Move Specs one dependency level.
void launch_fill_bounded(const DevParams* P, int mode, bool units, const uint32_t* all_level_shapes, const BoundSegs& segs, uint64_t* cost,
                         uint16_t* arg, Counters* ctr, hipStream_t stream) {
  if (!segs.n || !segs.block0[segs.n]) return;
  const dim3 grid(segs.block0[segs.n]);
  const bool two = segs.lanes_per_wave >= 128;
  if (mode == 1 && two) hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_units_kernel<1, 2>), grid, dim3(256), 0, stream, P, all_level_shapes, segs, cost, arg, ctr);
  else if (mode == 1) hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_units_kernel<1, 1>), grid, dim3(256), 0, stream, P, all_level_shapes, segs, cost, arg, ctr);
  else if (units && two) hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_units_kernel<0, 2>), grid, dim3(256), 0, stream, P, all_level_shapes, segs, cost, arg, ctr);
  else if (units) hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_units_kernel<0, 1>), grid, dim3(256), 0, stream, P, all_level_shapes, segs, cost, arg, ctr);
  else hipLaunchKernelGGL(fill_bounded_kernel, grid, dim3(256), 0, stream, P, all_level_shapes, segs, cost, arg, ctr);
}

// (a lane's offset inside a unit is 32 bits of bytes)
bool fill_by_units(int mode, uint64_t qv) { return mode == 1 || (mode == 0 && qv >= kUnitLanes && qv < (1ull << 29)); }

// ---------------------------------------------------------------- launches
uint32_t unit_blocks(const uint32_t* level_off, uint32_t n_levels, uint32_t npass, uint32_t* blk_off) {
  uint32_t n = 0;
  for (uint32_t l = 0; l < n_levels; l++) {
    if (blk_off) blk_off[l] = n;
    n += ((level_off[l + 1] - level_off[l]) * npass + kBlockItems - 1) / kBlockItems;
  }
  if (blk_off) blk_off[n_levels] = n;
  return n;
}
// (Refused: a level of 2^28 items and more, with Move Specs 2^27, and 2^30 shapes.  The plan takes a lane per item, in blocks of eight; the scan a workgroup
// per level and rank, in whose last one a lane of a wave is a diagonal.)
bool plan_fits(const DevParams& h, uint32_t n_shapes, const uint32_t* level_off, uint32_t n_levels) {
  if (n_shapes >= (1u << 30) - 64u || n_levels > kMaxLevels - kMaxRanks + 1) return false;
  for (uint32_t l = 0; l < n_levels; l++)
    if ((uint64_t)(level_off[l + 1] - level_off[l]) * h.npass >= (1ull << 32) / (h.moves ? 32 : 16)) return false;
  return true;
}
size_t plan_bytes_recs(uint32_t n_shapes) { return (size_t)n_shapes * sizeof(ShapeRec); }

void launch_plan(const DevParams* P, const DevParams& h, uint32_t n_levels, uint32_t n_blk, const PlanBuffers& B, Counters* ctr, hipStream_t stream) {
  hipLaunchKernelGGL(plan_kernel, dim3((uint32_t)(((uint64_t)n_blk * kBlockItems + 255) / 256)), dim3(256), 0, stream, P, B.level_shapes, B.level_off, B.blk_off, n_levels, n_blk,
                     (ShapeRec*)B.recs, B.masks, B.cnt);
  hipLaunchKernelGGL(scan_units_kernel, dim3(n_levels * h.nranks), dim3(1024), 0, stream, B.blk_off, n_levels, h.nranks, n_blk, B.cnt, B.seg, B.host_diag, &ctr->ticket);
}

void launch_fit_map(const DevParams* P, uint32_t n_specs, const PlanBuffers& B, uint32_t* fitmap, uint32_t n_words, hipStream_t stream) {
  hipLaunchKernelGGL(fit_map_kernel, dim3((n_words + 2 + 255) / 256), dim3(256), 0, stream, P, n_specs, B.masks, (unsigned long long*)fitmap, n_words);
}

void launch_list_units(const DevParams* P, const DevParams& h, uint32_t n_levels, const uint32_t* h_blk_off, const PlanBuffers& B, uint32_t w0, uint32_t w_len, uint32_t d0, uint32_t d1,
                       uint64_t none_from, hipStream_t stream) {
  const uint32_t n_blk = h_blk_off[n_levels];
  const uint64_t items = (uint64_t)n_blk * kBlockItems;
  uint32_t each = h.ncombo > 64 ? kListItems / 4 : kListItems;      // (enough workgroups, of a few hundred units)
  while (each > 64 && items / each * h.nranks < 2048) each /= 2;
  // the levels that have units of a rank on diagonals d0 to d1
  ListFirst firsts;
  uint32_t most = 0;
  for (uint32_t r = 0; r < kMaxRanks; r++) {
    const uint32_t l0 = d0 > r ? d0 - r : 0, l1 = d1 < r ? 0 : std::min(d1 - r + 1, n_levels);
    firsts.block[r] = n_blk;
    if (r >= h.nranks || l0 >= l1) continue;
    firsts.block[r] = h_blk_off[l0];
    most = std::max(most, h_blk_off[l1] - h_blk_off[l0]);
  }
  hipLaunchKernelGGL(list_units_kernel, dim3((uint32_t)(((uint64_t)most * kBlockItems + each - 1) / each), h.nranks), dim3(256), 0, stream, P, B.level_shapes, B.level_off, B.blk_off, n_levels, n_blk,
                     (const ShapeRec*)B.recs, B.masks, B.cnt, B.seg, (uint2*)B.list, w0, w_len, each, (uint32_t)std::min<uint64_t>(none_from, UINT32_MAX), firsts);
}

void launch_bind(const DevParams* P, uint64_t* bind, uint32_t n, hipStream_t stream) {
  hipLaunchKernelGGL(bind_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, P, bind, n);
}

FillArgs fill_args(const DevParams* d_P, const DevParams& h, const PlanBuffers& B, uint64_t* cost, uint16_t* arg, Counters* ctr) {
  FillArgs A;
  memset(&A, 0, sizeof A);
  A.P = d_P; A.recs = B.recs; A.steps = h.steps; A.cost = cost; A.arg = arg; A.ctr = ctr;
  A.costM = h.costM; A.costE = h.costE; A.mk_entry = h.mk_entry;
  A.nranks = h.nranks; A.npass = h.npass; A.nwp = h.nwp; A.nops = h.nops; A.NL = h.NL; A.G = h.G; A.log2V = h.log2V; A.ndt = h.ndt;
  for (uint32_t i = 0; i < 4; i++) {
    A.mstride[i] = h.mstride[i]; A.pack_shift[i] = h.pack_shift[i]; A.lay_bit[i] = h.lay_bit[i];
    A.lay_xor[i] = i < h.nops && h.lay_bit[i] != kNoBit ? 1u << h.lay_bit[i] : 0u;
    A.cv_bit[i] = i < h.nops && h.can_convert[i] && h.dt_bit[i] != kNoBit ? 1u << h.dt_bit[i] : 0u;
    A.zero[i] = h.zero[i];
  }
  A.unit_lay = h.unit_lay; A.lg_split = lg_split_lanes(h.moves || h.nlay); A.convert = h.convert; A.s = h.s; A.sync = h.sync;
  A.move_base = h.move_base; A.buf_id = h.buf_id; A.par_shift = h.par_base - h.tile_base;
  A.has_buf = h.kind == kKindF || h.split; A.split = h.split; A.chain = h.chain;
  A.GM = h.GM; A.VM = h.VM; A.GE = h.GE; A.VE = h.VE; A.nszE_n = h.nszE_n; A.kM_first = h.kM_first; A.nkM = h.nkM; A.nsz3 = h.nsz[3];
  for (int i = 0; i < 3; i++) { A.layM[i] = h.layM[i]; A.layE[i] = h.layE[i]; }
  return A;
}

// Which kernel takes a diagonal.  Split entries have short chains of reads, which is what counts while the chip is not full; the
// others issue fewer instructions per entry (diagonals of 20 blocks of a lane per entry 20 us, split 5; of 1.6 M entries, four
// at a time, 33, a lane each 61, split more).  The line at 16,384, 32,768 or 65,536 entries: within 1 % of each other; none split: the
// vector-matrix product 485 -> 594 us, the pipeline 3082 -> 3109; all split: 3912, two Matmuls 2001 -> 3196, packed layouts 2397 -> 2922.
// Without layouts (four lanes) a Matmul's split is never behind: all sizes to 64, 668 against 740 us of fill; where m and n alone are tiled and the
// bufferize is one lane's, it is: fused, sizes to 40 and 48, alone, all split 2098 and 3131 us, the line at 131,072 entries 1953 and 2923; at 32,768 the
// same, but the pipeline's sizes to 256 1236 -> 1269.  With parallel loops, three layouts, sizes to 24 and 40 of which much fits: four at a time from 32,768
// entries 802 and 1560 us, from 262,144 819 and 1583 (a lane each instead of four at a time, from 262,144: 998 and 1966).
template <bool LAY, bool MOVES, bool SMALL, bool PAR, bool MN>
static void launch_run(const FillArgs& A, const uint2* list, const DiagRun& run, hipStream_t stream) {
  const uint32_t n = run.start[1] - run.start[0];
  const uint64_t tasks = (uint64_t)n << A.unit_lay;
  const uint2* units = list + run.start[0];
  const auto blocks = [](uint64_t lanes) { return dim3((uint32_t)((lanes + 255) / 256)); };
  if (run.chain) hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_chain_kernel<LAY, MOVES, SMALL, PAR, MN>), dim3(1), dim3(kChainThreads), 0, stream, A, list, run);
  else if ((!LAY && !MN) || tasks <= (LAY ? kSplitTasks : kBareSplitTasks))
    hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_split_kernel<LAY, MOVES, SMALL, PAR, MN>), blocks(tasks << A.lg_split), dim3(256), 0, stream, A, units, n);
  else if constexpr (LAY || MN) {
    if constexpr (LAY && !MOVES)
      if (!A.ndt && A.unit_lay >= 2) {
        hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_quad_kernel<SMALL, PAR, MN>), blocks(tasks), dim3(256), 0, stream, A, units, n);
        return;
      }
    hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_entry_kernel<MOVES, SMALL, PAR, MN>), blocks(tasks), dim3(256), 0, stream, A, units, n);
  }
}

// From how many units on the levels of shapes are filled at once (fill_shapes_kernel) instead of by diagonals.  A launch of a level takes some 25 us, through
// tiles and ranks, a small diagonal 6; a place of a shape that does not fit is a lane that idles; in return a unit is shorter, for the groups of a shape
// and of its tiles are read once, not once for each rank.  So: as many as units_for_a_launch for each level, and a part of all places: a larger one the more layouts, which
// the diagonals take four at a time (fill_quad_kernel) and the levels one by one.  Both fitted to ten tables and more of each form, of three sizes, of
// which 10 to 100 % fits; solve alone, by diagonals and by levels, in us, on either side of the line.  A Matmul of all sizes to 56: 48 % 1096 and 1042, 30 % 922 and 1012; to
// 80: 30 % 2674 and 2528, 17 % 1944 and 2164; to 36, everything: 685 and 735.  One layout, to 56: 1509 and 1424, 1168 and 1288; two: 70 % 2585 and
// 2320, 48 % 2031 and 2144; three: everything 5328 and 4505, 70 % 4137 and 4244, to 80, 30 % 12267 and 14227.  A dtype bit, to 60: 35 % 1418 and
// 1240, 18 % 989 and 1115.  Parallel loops, to 60: 44 % 1573 and 1447, 27 % 1229 and 1393; three layouts, to 44: 85 % 3048 and 2915, 63 % 2412 and 2642.
// Fused, to 40: 38 % 3316 and 2995, 15 % 1866 and 2269; two Matmuls composed, to 6, everything 414 and 389, to 4 332 and 347; bias add, ReLU and the two, to 255,
// everything 2087 and 1870, to 160 1345 and 1559.
// (Move Specs' prices are a table of their own, and fused Specs with layouts have more cells than a workgroup takes.)
// Where the scratch holds a part of the work list at a time, every further part is a launch between two others, 14 to 24 us (alone, bias add and
// ReLU, to 255, 5 dependency levels: ample scratch 914 us, 64 parts 2451, by levels 761): it counts as a level does.
uint32_t units_for_a_launch(const DevParams& h) {
  return h.chain ? 200000 : h.npass > 1 ? 340000 : h.kind != kKindM ? 150000 : h.ndt ? 220000 : h.par ? (h.nlay ? 110000 : 160000) : h.nlay ? 150000 : 190000;
}
uint64_t by_shapes_from(const DevParams& h, uint32_t n_shapes, uint32_t n_levels) {
  if (h.moves || (h.nlay && h.kind != kKindM) || h.G > kShapeCells || h.G <= (h.nlay ? 64u : 32u)) return UINT64_MAX;
  const uint64_t places = ((uint64_t)n_shapes * h.npass * h.ncombo) << h.ndt;
  const uint64_t percent = h.kind != kKindM ? 22 : h.nlay == 0 ? 16 : h.nlay == 1 ? 19 : h.nlay == 2 ? 33 : 50;
  return std::max(kShapeUnits, (uint64_t)units_for_a_launch(h) * n_levels + places * percent / 100);
}
void launch_fill_shapes(const FillArgs& A, const DevParams& h, const unsigned long long* masks, uint32_t first, uint32_t n, hipStream_t stream) {
  uint32_t lg_cells = 0, lg_lanes = 0, most = 0;
  while ((1u << lg_cells) < h.G) lg_cells++;
  for (uint32_t r = 0; r < h.nranks; r++) most = std::max(most, (h.rank_off[r + 1] - h.rank_off[r]) << h.log2V);
  while (lg_lanes < 6 && (1u << lg_lanes) < most) lg_lanes++;
  const uint32_t each = kShapeCells >> lg_cells;
  RankOff ranks;
  for (uint32_t r = 0; r < kMaxRanks + 2; r++) ranks.at[r] = (uint16_t)h.rank_off[r];
  const dim3 grid((n + each - 1) / each);
#define MRL_SHAPES(lay, par, mn) do { \
    if (h.small) hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_shapes_kernel<lay, true, par, mn>), grid, dim3(256), 0, stream, A, ranks, (const ShapeRec*)A.recs, A.steps, masks, first, n, lg_cells, lg_lanes); \
    else hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_shapes_kernel<lay, false, par, mn>), grid, dim3(256), 0, stream, A, ranks, (const ShapeRec*)A.recs, A.steps, masks, first, n, lg_cells, lg_lanes); \
  } while (0)
  if (h.par && h.nlay) MRL_SHAPES(true, true, false);
  else if (h.par) MRL_SHAPES(false, true, false);
  else if (h.kind != kKindM) MRL_SHAPES(false, false, true);
  else if (h.nlay) MRL_SHAPES(true, false, false);
  else MRL_SHAPES(false, false, false);
#undef MRL_SHAPES
}

bool small_diagonal(const FillArgs& A, uint32_t n) { return (uint64_t)n << (A.unit_lay + A.lg_split) <= kChainThreads; }

// (a launch has fewer than 2^32 threads, in workgroups of 256; split entries have the most)
uint32_t most_units(const FillArgs& A) { return (uint32_t)(((1ull << 32) - 256) >> (A.unit_lay + A.lg_split)); }

void launch_fill_diagonals(const FillArgs& A, const DevParams& h, const void* list, const DiagRun& run, hipStream_t stream) {
  const uint2* l = (const uint2*)list;
  const bool mn = h.kind != kKindM;
#define MRL_RUN(lay, moves, par, mn) (h.small ? launch_run<lay, moves, true, par, mn>(A, l, run, stream) : launch_run<lay, moves, false, par, mn>(A, l, run, stream))
  if (h.moves) MRL_RUN(true, true, false, false);
  else if (h.par && h.nlay) MRL_RUN(true, false, true, false);
  else if (h.par) MRL_RUN(false, false, true, false);
  else if (mn && h.nlay) MRL_RUN(true, false, false, true);
  else if (mn) MRL_RUN(false, false, false, true);
  else if (h.nlay) MRL_RUN(true, false, false, false);
  else MRL_RUN(false, false, false, false);
#undef MRL_RUN
}

}  // namespace mrl
