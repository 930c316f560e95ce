// Rewrite evaluation + argmin for one dependency level of the Spec lattice.
//
// Paper, Section 4: a Spec's entry is the lowest-cost applicable rewrite, the
// rewrite's cost being the affine function of Section 3 of its sub-Specs'
// costs.  Here the table is filled bottom-up: all shapes of one dependency
// level in one launch, every sub-Spec of another shape already final.
//
// An item is one shape (b,m,k,n) at one value of the passive level axis (the
// intermediate's level of a fused Spec; other kinds have one value): a set of
// entries closed under Moves.  Before the first level a plan kernel decides,
// for every item and every value of the dtype bits, which level assignments
// fit their levels (most do not), as one bit mask per item in rank order
// (rank = sum of the operand levels), and sets the whole table to (INF, NONE),
// so that the level kernels write admissible entries only; a second kernel
// puts the items with anything to do into work lists per dependency level:
// bundles of items (about kBundle tasks together; a task is an admissible
// entry) and wide items of their own.
//
// A workgroup takes a bundle.  Its first lanes take an item each (shape,
// masks, tile counts, everything that does not depend on the entry), then the
// admissible entries of all its items are listed in LDS, once by item and once
// by rank, and
//   1. one lane per task evaluates the tile and bufferize rewrites, whose
//      sub-Specs belong to other shapes or tables and are final: a tile
//      sub-Spec sits at the same offset of a smaller shape's group, several
//      loads in flight per lane.  The best of them is parked in LDS;
//   2. rank by rank, a quad of lanes per task evaluates the Moves (sub-Specs
//      of the same item at a lower rank: read from LDS), an operand per lane;
//      the quad's first lane adds the microkernels and the parked candidate;
//   3. the results go to the table, a task per lane.
// The ranks of a shape are a chain (10 of three operands, 13 of four), and a
// rank of one item holds only a few tasks; the bundle's items go through it
// together, which fills the lanes, and share the cost of setting up.
// Ties go to the lowest id: a lane meets its candidates in the order of their
// ids where it compares the cost alone, all else is compared by (cost, id).
// Nothing is reduced across workgroups: the table is deterministic.
#include <hip/hip_runtime.h>
#include "compress.h"
#include "dev_params.h"

namespace mrl {

constexpr int kBatch = 8;              // sub-Spec costs fetched together before they are compared

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
  const uint64_t b = S.d[0], m = S.d[1], k = S.d[2], n = S.d[3];
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

// What the level kernels need of a shape, worked out once by the plan kernel.
struct alignas(16) ShapeRec {
  uint64_t numel[5];             // elements of the operands ([4]: the intermediate)
  uint32_t shape, si;            // index; the four size indices, a byte each
  uint32_t n_serial, n_tile;     // tile rewrites: serial loops, with parallel loops
  uint32_t tile_lo[4], tile_cnt; // first entry of each dimension's list of tiles, their numbers (a byte each)
  uint32_t mk_var;               // microkernels whose shape predicate holds (bits 0..7); packed layouts: layouts that exist << 8 (see variant_of)
};
static_assert(sizeof(ShapeRec) == 80, "read as five 16-byte pieces");

// Plan: one wave per up to kPlanShapes shapes, in the order of the dependency levels.  Its first lanes take
// a shape each and write its record; then, shape by shape, the lanes are level assignments: which
// of them fit is written as one mask per item (bit = position in rank order, one plane of nwp words
// per value of the dtype bits) with the item's number of tasks, and the entries that fit are marked
// in a bit map in table order (bit = cell; read by the compression pass).
// Bound by instruction issue (460 vector instructions a shape), on small tables by the latency of a wave's shapes one
// after the other: with 16 per wave always, config 3's 180 shapes took 46 us, now 11.  The map is stored whole where
// that can be done: with an atomic per level assignment config 2 (262,144 shapes, one bit each) took 178 us, now 129.
constexpr uint32_t kPlanShapes = 16, kPlanWaves = 4096;      // shapes per wave at most, and fewer while there are fewer waves than this
// Whether the plan stores the map whole (a level assignment's bits, passive levels x variants, are a power of two of
// them, and those of all level assignments whole bytes); else it adds bits to a map that is zero before.
bool fit_map_stored(const DevParams& h) {
  const uint32_t nb = h.npass * h.V;
  return (nb & (nb - 1)) == 0 && (nb >= 8 || (h.ncombo <= 64 && h.ncombo * nb % 8 == 0));
}
static uint32_t plan_shapes(uint32_t n_shapes) {
  uint32_t per = kPlanShapes;
  while (per > 1 && n_shapes / per < kPlanWaves) per /= 2;
  return per;
}

__global__ __launch_bounds__(256) void plan_kernel(const DevParams* __restrict__ P, uint32_t n_shapes, uint32_t per_wave, uint32_t map_stored, const uint32_t* __restrict__ level_shapes,
                                                   ShapeRec* __restrict__ recs, unsigned long long* __restrict__ masks,
                                                   uint16_t* __restrict__ item_tasks, uint32_t* __restrict__ fitmap, Counters* __restrict__ ctr,
                                                   uint4* __restrict__ cost16, uint4* __restrict__ arg16) {
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t npass = P->npass, ncombo = P->ncombo, V = P->V, nb = npass * V, ndp = 1u << P->ndt, nwp = P->nwp, nw = ndp * nwp, NL = P->NL, nops = P->nops;
  const uint32_t first = (blockIdx.x * 4 + wave) * per_wave;
  if (first >= n_shapes) return;
  const uint32_t n_here = n_shapes - first < per_wave ? n_shapes - first : per_wave;
  // ---- a shape per lane ----
  Shape S;
  uint32_t shape = 0, var = 0, nvb = 0;
  unsigned long long lays = 1;                  // bit v: variant v (dtype bits 0) has layouts that exist
  if (lane < n_here) {
    shape = level_shapes[first + lane];
    load_shape(P, shape, S);
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
    for (uint32_t i = nops; i-- > 0;) {         // from the lowest layout field up
      const uint32_t w = layout_width(P, S, i);
      if (i < 3) var |= w << (2 * i) | nvb << (8 + 4 * i);
      nvb += w;
      if (!w) continue;
      const uint32_t step = 1u << P->lay_bit[i];
      lays |= lays << step;
      if (w == 2) lays |= lays << (2 * step);
    }
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
    uint4* to = reinterpret_cast<uint4*>(recs + first + lane);
#pragma unroll
    for (int i = 0; i < 5; i++) to[i] = from[i];
  }
  // ---- a level assignment per lane ----
  uint32_t info[4], off0[4];
#pragma unroll
  for (int it = 0; it < 4; it++) {
    info[it] = it * 64 + lane < ncombo ? P->pos_info[it * 64 + lane] : 0u;
    off0[it] = it * 64 + lane < ncombo ? ((P->pos_entry[it * 64 + lane] >> 16) * npass) << P->log2V : 0u;      // pass 0, variant 0 of this level assignment
  }
  const bool fused = P->kind == kKindF;
  unsigned long long n_adm = 0;
  for (uint32_t s = 0; s < n_here; s++) {
    const uint32_t sh = lane_of(shape, s), vb = lane_of(nvb, s);
    const unsigned long long lay_s = (unsigned long long)lane_of((uint32_t)(lays >> 32), s) << 32 | lane_of((uint32_t)lays, s);
    uint64_t numel[5];
#pragma unroll
    for (int i = 0; i < 5; i++) numel[i] = (uint64_t)lane_of((uint32_t)(S.numel[i] >> 32), s) << 32 | lane_of((uint32_t)S.numel[i], s);
    if (cost16) {
      // (INF, NONE) = all-ones over the shape's whole group: the level kernels overwrite what fits
      const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u);
      const uint32_t nc = P->G >> 1, na = P->G >> 3;       // 16-byte pieces (G is a multiple of 8)
      uint4* c16 = cost16 + (size_t)sh * nc;
      uint4* a16 = arg16 + (size_t)sh * na;
      for (uint32_t i = lane; i < nc; i += 64) c16[i] = ones;
      for (uint32_t i = lane; i < na; i += 64) a16[i] = ones;
    }
    const uint64_t group = (uint64_t)sh * P->G;
    uint32_t ents[4] = {0, 0, 0, 0};
    unsigned long long my_word = 0;             // lane pass * nw + word keeps that word
    unsigned long long bits[4] = {0, 0, 0, 0};
    for (uint32_t dt = 0; dt < ndp; dt++) {
      // bit b of fit[l]: the tensors of subset b (operands 0..3, bit 4 = the intermediate) together fit level l
      uint64_t sum = 0;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        if ((uint32_t)i >= nops) break;
        const uint32_t bf = P->dt_bit[i] != kNoBit ? (dt >> P->dt_bit[i]) & 1u : P->base_bf16[i];
        sum += (lane >> i) & 1u ? numel[i] << (bf ? 1u : 2u) : 0;
      }
      sum += (lane >> 4) & 1u ? numel[4] << 2 : 0;
      uint32_t fit[4];
#pragma unroll
      for (int l = 0; l < 4; l++) fit[l] = (uint32_t)__ballot(sum <= P->cap[l]);
#pragma unroll
      for (int it = 0; it < 4; it++) {
        if ((uint32_t)(it * 64) >= ncombo) break;
#pragma unroll
        for (int ps = 0; ps < 4; ps++) {
          if ((uint32_t)ps >= npass) break;
          uint32_t ok = it * 64 + lane < ncombo ? 1u : 0u;
#pragma unroll
          for (int l = 0; l < 4; l++)
            if ((uint32_t)l < NL) ok &= fit[l] >> (((info[it] >> (8 + 4 * l)) & 15u) | (fused && ps == l ? 16u : 0u));
          const unsigned long long bal = __ballot(ok & 1u);
          if (lane == ps * nw + dt * nwp + it) my_word = bal;
          ents[ps] += (uint32_t)__popcll(bal);
          if (ok & 1u) bits[it] |= lay_s << (dt + ps * V);
        }
      }
    }
    if (nb < 8 && map_stored) {
      // less than a byte per level assignment: the lanes go from rank to table order, and as many as make a byte join up
      uint32_t x = (uint32_t)__builtin_amdgcn_ds_permute((int)(lane < ncombo ? off0[0] / nb : lane) * 4, (int)(uint32_t)bits[0]);
      for (uint32_t have = nb, d = 1; have < 8; have *= 2, d *= 2) x |= (uint32_t)__shfl_down((int)x, d, 64) << have;
      if (lane * nb % 8 == 0 && lane < ncombo) ((uint8_t*)fitmap)[(group + lane * nb) >> 3] = (uint8_t)x;
    } else {
#pragma unroll
      for (int it = 0; it < 4; it++) {
        if ((uint32_t)(it * 64) >= ncombo) break;
        if (it * 64 + lane >= ncombo) continue;
        const uint64_t cell0 = group + off0[it];
        if (map_stored) {
          // whole bytes to pairs of words (the group size is a multiple of nb): stored, the map is not zeroed
          if (nb == 8) ((uint8_t*)fitmap)[cell0 >> 3] = (uint8_t)bits[it];
          else if (nb == 16) ((uint16_t*)fitmap)[cell0 >> 4] = (uint16_t)bits[it];
          else {
            fitmap[cell0 >> 5] = (uint32_t)bits[it];
            if (nb == 64) fitmap[(cell0 >> 5) + 1] = (uint32_t)(bits[it] >> 32);
          }
        } else if (bits[it]) {
          const uint32_t shift = (uint32_t)(cell0 & 31u);
          uint32_t* w = fitmap + (cell0 >> 5);
          atomicOr(w, (uint32_t)(bits[it] << shift));
          if (shift + nb > 32) {
            atomicOr(w + 1, (uint32_t)(bits[it] >> (32 - shift)));
            if (shift + nb > 64) atomicOr(w + 2, (uint32_t)(bits[it] >> (64 - shift)));
          }
        }
      }
    }
    if (lane < npass * nw) masks[(size_t)(first + s) * npass * nw + lane] = my_word;
    const uint32_t mine = lane == 0 ? ents[0] : lane == 1 ? ents[1] : lane == 2 ? ents[2] : ents[3];
    if (lane < npass) item_tasks[(size_t)(first + s) * npass + lane] = (uint16_t)(mine << vb);
    n_adm += (unsigned long long)(ents[0] + ents[1] + ents[2] + ents[3]) << vb;
  }
  if (lane == 0 && n_adm) atomicAdd(&ctr->n_admissible[blockIdx.x % kCtrSlots], n_adm);
}

// Work lists, kSortTile items of one dependency level per workgroup: the level's items in order,
// those of at most small_max tasks cut into bundles (bundle b = items [bundle_first[b],
// bundle_first[b + 1]) of the level's stretch of list_small), the others in list_wide.  An item
// weighs its tasks (at least min_weight, which bounds the items of a bundle); a bundle ends with the
// item that fills its quota, kBundle tasks on levels with work enough to fill the chip, less on
// others.  Levels of several tiles: sort_sums_kernel first adds up every tile.
constexpr uint32_t kSortThreads = 1024, kSortItems = 8, kSortTile = kSortThreads * kSortItems;
// (sweeps with the final kernels: quotas of 64, 96, 192 and 256 tasks are 0 to 3 % slower on the
// large lattices, 2048 and 4096 bundles before they grow 3 and 8 % on config 4, 512 the same)
constexpr uint32_t kBundle = 128;            // tasks per bundle
constexpr uint32_t kFewBundles = 256, kManyTasks = 7;      // a bundle has a compute unit for itself, and 2^7 tasks and more
constexpr uint32_t kMinBundles = 1024;       // a level is cut into this many bundles before they grow

__device__ __forceinline__ unsigned long long block_scan_1024(unsigned long long v, unsigned long long* sh, unsigned long long& total) {
  unsigned long long incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned long long o = __shfl_up(incl, d, 64);
    if ((int)(threadIdx.x & 63u) >= d) incl += o;
  }
  __syncthreads();
  if ((threadIdx.x & 63u) == 63) sh[threadIdx.x >> 6] = incl;
  __syncthreads();
  unsigned long long excl = incl - v;
  total = 0;
  for (uint32_t w = 0; w < kSortThreads / 64; w++) {
    const unsigned long long x = sh[w];
    if (w < (threadIdx.x >> 6)) excl += x;
    total += x;
  }
  return excl;
}

// The level and the tile of it that workgroup `b` has: levels in order, each with its tiles.
__device__ __forceinline__ void sort_place(const uint32_t* __restrict__ level_off, uint32_t npass, uint32_t b, uint32_t& lv, uint32_t& tile) {
  lv = 0;
  tile = b;
  for (;;) {
    const uint32_t t = ((level_off[lv + 1] - level_off[lv]) * npass + kSortTile - 1) / kSortTile;
    if (tile < t) return;
    tile -= t;
    lv++;
  }
}

// sums[workgroup]: tasks of the tile's small items.
__global__ __launch_bounds__(kSortThreads) void sort_sums_kernel(const uint32_t* __restrict__ level_off, uint32_t npass, const uint16_t* __restrict__ item_tasks,
                                                                 uint32_t small_max, uint32_t* __restrict__ sums) {
  __shared__ unsigned long long sh[kSortThreads / 64];
  uint32_t lv, tile;
  sort_place(level_off, npass, blockIdx.x, lv, tile);
  const uint32_t first = level_off[lv] * npass, n = (level_off[lv + 1] - level_off[lv]) * npass, base = tile * kSortTile;
  unsigned long long work = 0, total = 0;
  for (uint32_t i = base + threadIdx.x; i < n && i < base + kSortTile; i += kSortThreads) { const uint32_t t = item_tasks[first + i]; if (t <= small_max) work += t; }
  block_scan_1024(work, sh, total);
  if (threadIdx.x == 0) sums[blockIdx.x] = (uint32_t)total;
}

// part 0: with the quota known, the weights and numbers of the tile (parts[workgroup]); part 1: the
// lists.  A grid of one tile per level needs part 1 only.
__global__ __launch_bounds__(kSortThreads) void sort_work_kernel(const uint32_t* __restrict__ level_off, uint32_t n_levels, uint32_t npass,
                                                                 const uint16_t* __restrict__ item_tasks, uint32_t small_max, uint32_t min_weight,
                                                                 uint32_t part, const uint32_t* __restrict__ sums, uint4* __restrict__ parts,
                                                                 uint32_t* __restrict__ list_small, uint32_t* __restrict__ bundle_first,
                                                                 uint32_t* __restrict__ list_wide, uint32_t* __restrict__ list_cnt) {
  __shared__ unsigned long long sh[kSortThreads / 64];
  uint32_t lv, tile;
  sort_place(level_off, npass, blockIdx.x, lv, tile);
  const uint32_t first = level_off[lv] * npass, n = (level_off[lv + 1] - level_off[lv]) * npass, base = tile * kSortTile;
  const uint32_t tiles = (n + kSortTile - 1) / kSortTile, wg0 = blockIdx.x - tile;
  uint32_t tasks[kSortItems];
  unsigned long long work = 0, total = 0;
#pragma unroll
  for (uint32_t k = 0; k < kSortItems; k++) {
    const uint32_t i = base + threadIdx.x * kSortItems + k;
    tasks[k] = i < n ? item_tasks[first + i] : 0u;
    if (tasks[k] <= small_max) work += tasks[k];
  }
  if (sums) for (uint32_t t = 0; t < tiles; t++) total += sums[wg0 + t];
  else block_scan_1024(work, sh, total);
  const uint32_t level_tasks = (uint32_t)total;
  uint32_t quota = (uint32_t)(total / kMinBundles);
  quota = quota < min_weight ? min_weight : quota > kBundle ? kBundle : quota;
  auto weight = [&](uint32_t t) { return t < min_weight ? min_weight : t > quota ? quota : t; };
  unsigned long long mine = 0;                      // weight (32 bits) | small items (16) | wide items (16)
#pragma unroll
  for (uint32_t k = 0; k < kSortItems; k++) {
    if (tasks[k] > small_max) mine += 1ull << 48;
    else if (tasks[k]) mine += 1ull << 32 | weight(tasks[k]);
  }
  const unsigned long long excl = block_scan_1024(mine, sh, total);
  const uint32_t all_w = (uint32_t)total, all_s = (uint32_t)((total >> 32) & 0xFFFFu), all_x = (uint32_t)(total >> 48);
  if (part == 0) {
    if (threadIdx.x == 0) parts[blockIdx.x] = make_uint4(all_w, all_s, all_x, 0);
    return;
  }
  uint32_t run_w = 0, run_s = 0, run_x = 0;          // weight and number of the small items, number of the wide ones, of the tiles before
  if (sums)
    for (uint32_t t = 0; t < tile; t++) { const uint4 p = parts[wg0 + t]; run_w += p.x; run_s += p.y; run_x += p.z; }
  uint32_t w = run_w + (uint32_t)excl, s = run_s + (uint32_t)((excl >> 32) & 0xFFFFu), x = run_x + (uint32_t)(excl >> 48);
  uint32_t* starts = bundle_first + first + lv;
#pragma unroll
  for (uint32_t k = 0; k < kSortItems; k++) {
    const uint32_t item = first + base + threadIdx.x * kSortItems + k;
    if (tasks[k] > small_max) list_wide[first + x++] = item;
    else if (tasks[k]) {
      const uint32_t add = weight(tasks[k]);
      list_small[first + s++] = item;
      if ((w + add) / quota != w / quota) starts[(w + add) / quota] = s;       // (weights are at most the quota: no bundle is skipped)
      w += add;
    }
  }
  if (threadIdx.x == 0) {
    if (tile == 0) starts[0] = 0;
    if (tile + 1 == tiles) {
      const uint32_t bundles = (run_w + all_w + quota - 1) / quota;
      starts[bundles] = run_s + all_s;
      const uint32_t each = bundles ? level_tasks / bundles : 0u, lg = each ? 31u - (uint32_t)__builtin_clz(each) : 0u;
      list_cnt[lv] = bundles; list_cnt[n_levels + lv] = run_x + all_x;
      list_cnt[2 * n_levels + lv] = (run_s + all_s) | (lg < 15u ? lg : 15u) << kItemsBits;       // (plan_fits: fewer than 2^28 items)
    }
  }
}

// ---------------------------------------------------------------- one dependency level
// LDS of a workgroup: up to cap tasks of up to ni items, kt tile rewrites per item at a time.
struct FillGeom {
  uint32_t cap, ni, kt;
  uint32_t bt;          // Move-cost entries per item
  uint32_t isz;         // entries of an item's table of level assignments (dtype bits x pack)
  uint32_t nlay;        // layout bits; without MOVES a task index is an entry index and these bits
  uint32_t ns;          // entries at most; entry ns stands for "does not fit" (its tasks cost INF)
};

struct FillLds {
  uint64_t *t_cost, *bterm, *it_numel, *it_z;
  unsigned long long* it_mask;
  uint32_t *tl_cell, *tl_trips, *tl_id, *ent, *rl_ent, *it_base, *it_si, *it_pass, *it_ntile, *it_nserial, *it_first, *it_mk, *it_rowM, *it_rowE, *it_var, *it_lo, *it_cnt, *rcnt;
  uint16_t *t_arg, *rl_slot, *place, *idx, *tk0, *tslot;
};

// Carves the workgroup's LDS (w = nullptr: only counts the bytes).
__host__ __device__ inline uint32_t carve_fill(unsigned char* w, const FillGeom& g, bool moves, FillLds& L) {
  uint32_t o = 0;
  auto take = [&](uint32_t bytes) { unsigned char* p = w + o; o += (bytes + 15u) & ~15u; return p; };
  L.t_cost = (uint64_t*)take((g.cap + (1u << g.nlay)) * 8);
  L.bterm = (uint64_t*)take(g.ni * g.bt * 8);
  L.it_numel = (uint64_t*)take(g.ni * 5 * 8);
  L.it_z = (uint64_t*)take(g.ni * 8);
  L.it_mask = (unsigned long long*)take(g.ni * 4 * 8);
  L.tl_cell = (uint32_t*)take(g.ni * g.kt * 4);
  L.tl_trips = (uint32_t*)take(g.ni * g.kt * 4);
  L.tl_id = (uint32_t*)take(g.ni * g.kt * 4);
  L.ent = (uint32_t*)take(g.ns * 4);
  L.rl_ent = (uint32_t*)take(g.ns * 4);
  uint32_t* it = (uint32_t*)take((g.ni * 15 + 1) * 4);
  L.it_base = it; L.it_si = it + g.ni; L.it_pass = it + 2 * g.ni; L.it_ntile = it + 3 * g.ni; L.it_nserial = it + 4 * g.ni;
  L.it_mk = it + 5 * g.ni; L.it_rowM = it + 6 * g.ni; L.it_rowE = it + 7 * g.ni; L.it_var = it + 8 * g.ni; L.it_cnt = it + 9 * g.ni;
  L.it_lo = it + 10 * g.ni; L.it_first = it + 14 * g.ni;
  L.rcnt = (uint32_t*)take((kMaxRanks + 2) * 4);
  L.t_arg = (uint16_t*)take(g.cap * 2);
  L.rl_slot = (uint16_t*)take(g.ns * 2);
  L.place = (uint16_t*)take(g.ns * 2);
  L.idx = (uint16_t*)take(g.ni * g.isz * 2);
  L.tk0 = (uint16_t*)take(moves ? (g.ns + 1) * 2 : 0);
  L.tslot = (uint16_t*)take(moves ? g.cap * 2 : 0);
  return o;
}

// An entry of the workgroup's list: level assignment, dtype bits, item, rank, mixed-radix index.
__device__ __forceinline__ uint32_t ent_pack(uint32_t e) { return e & 0xFFu; }
__device__ __forceinline__ uint32_t ent_dt(uint32_t e) { return (e >> 8) & 3u; }
__device__ __forceinline__ uint32_t ent_item(uint32_t e) { return (e >> 10) & 63u; }
__device__ __forceinline__ uint32_t ent_rank(uint32_t e) { return (e >> 16) & 15u; }
__device__ __forceinline__ uint32_t ent_combo(uint32_t e) { return e >> 20; }

// Variant of an entry's c-th task.  Without packed layouts c is the layout bits; with them an item
// lists only the layouts that exist: var holds, per operand, the width of its field (2 bits at 2 * i)
// and the field's position inside c (3 bits at 8 + 4 * i).
template <bool MOVES>
__device__ __forceinline__ uint32_t variant_of(const DevParams* __restrict__ P, uint32_t var, uint32_t c, uint32_t dt) {
  if (!MOVES) return c << P->ndt | dt;
  uint32_t v = dt;
#pragma unroll
  for (int i = 0; i < 3; i++) {
    const uint32_t w = (var >> (2 * i)) & 3u;
    if (w) v |= ((c >> ((var >> (8 + 4 * i)) & 7u)) & ((1u << w) - 1u)) << P->lay_bit[i];
  }
  return v;
}

// bufferize (FUSED): Matmul into the intermediate, then bias-add+ReLU out of it.  The composition
// of two Matmuls (Section 2.1): the first, (m, k, p), into the intermediate, then the second,
// (m, p, n), out of it; both are entries of the same Matmul table.  The bias-add + ReLU with its
// own bufferize: per level l in which the intermediate fits next to the operands that live there,
// the bias add into it plus the ReLU out of it.  rowM, rowE: the shape's first entries in the two
// tables; z: cost of initialising the intermediate; numel: the item's element counts.
// Returns the number of candidates evaluated.
__device__ __forceinline__ uint32_t task_bufferize(const DevParams* __restrict__ P, uint32_t rowM, uint32_t rowE, uint64_t z,
                                                   const uint64_t* numel, uint32_t pack, uint32_t pass, uint32_t v, Eval& e) {
  const uint32_t NL = P->NL;
  const auto level = [&](int i) { return (pack >> P->pack_shift[i]) & 3u; };
  const auto lay = [&](int i) { return P->lay_bit[i] != kNoBit ? (v >> P->lay_bit[i]) & 1u : 0u; };
  const auto at = [](uint32_t y, uint32_t bit) { return bit != kNoBit ? y << bit : 0u; };
  if (P->split) {
    const uint32_t l0 = level(0), l1 = level(1), l2 = level(2);
    const uint32_t va = at(lay(0), P->layM[0]), vr = at(lay(2), P->layE[1]);
    uint32_t cnt = 0;
    for (uint32_t l = 0; l < NL; l++) {
      const uint64_t bytes = 4u * (numel[2] + (l0 == l ? numel[0] : 0u) + (l1 == l ? numel[1] : 0u) + (l2 == l ? numel[2] : 0u));
      if (bytes > P->cap[l]) continue;
      const uint64_t ca = P->costM[rowM + ((l0 * NL + l1) * NL + l) * P->VM + va];
      const uint64_t cr = P->costE[rowE + (l * NL + l2) * P->VE + vr];
      if (ca != kInf && cr != kInf) {
        if (ca + cr >= kLimit) e.ovf = 1; else consider(e, ca + cr, P->buf_id + l);     // each below 2^62: no wrap
      }
      cnt++;
    }
    return cnt;
  }
  const uint32_t l0 = level(0), l1 = level(1), l2 = level(2), l3 = level(3);
  const uint32_t xm = ((l0 * NL + l1) * NL + pass) * P->VM + at(lay(0), P->layM[0]) + at(lay(1), P->layM[1]);
  const uint32_t xe = P->chain ? ((pass * NL + l2) * NL + l3) * P->VM + at(lay(2), P->layM[1]) + at(lay(3), P->layM[2])
                               : ((pass * NL + l2) * NL + l3) * P->VE + at(lay(3), P->layE[2]);
  const uint64_t cm = P->costM[rowM + xm], ce = (P->chain ? P->costM : P->costE)[rowE + xe];
  if (cm != kInf && ce != kInf) {
    const uint64_t sum = z + cm;          // each term <= 2^62: no wrap
    if (z >= kLimit || sum >= kLimit || sum + ce >= kLimit) e.ovf = 1; else consider(e, sum + ce, P->buf_id);
  }
  return 1;
}

// Exchange inside a quad of lanes (lane ^ 1, lane ^ 2) without going through LDS.
template <int CTRL>
__device__ __forceinline__ uint32_t quad_swap(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ void quad_min(Eval& e) {
  const uint32_t lo = quad_swap<CTRL>((uint32_t)e.best), hi = quad_swap<CTRL>((uint32_t)(e.best >> 32));
  const uint32_t id = quad_swap<CTRL>(e.arg);
  consider(e, (uint64_t)hi << 32 | lo, id);
}

__device__ __forceinline__ void flush_counters(Counters* __restrict__ ctr, uint32_t n_rw, uint32_t ovf) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) n_rw += __shfl_down(n_rw, d, 64);
  if ((threadIdx.x & 63u) == 0 && n_rw) atomicAdd(&ctr->n_rewrites[blockIdx.x % kCtrSlots], (unsigned long long)n_rw);
  if (ovf) atomicOr(&ctr->overflow, ovf);
}

// One bundle (starts: the level's bundle starts; nullptr: an item each) per workgroup of T threads.
// LAY: the lattice has layout bits.  MOVES: the Matmul whose Moves are Move Specs.
// Bound by instruction issue on levels with many items (counters: 1,890 vector lane-instructions per
// task in config 5's F, 3,250 in config 2; the vector units issue half of the time that the launches
// of 128 threads take) and by the chain of memory and LDS round trips on the others (a fifth of the
// time there; 9 us for one item of 4 tasks: records 2.4, lists 2, tiles 2.3, ranks 1.8).  Fill
// times against one item per wave without bundles or records: config 2 1.49 -> 0.77 ms, config 3
// 0.69 -> 0.60, config 4 0.80 -> 0.73, config 5's F 2.22 -> 2.12, config 12's Matmul, which then was
// a lane per Spec with three gathers per Move, 5.04 -> 2.16.
// T: 512 for a wide item (100 registers would leave 2 instead of 3 workgroups on a unit, hence the
// bound), 256 on levels short of bundles, else 128 (64: config 4 +9 %, F +5 %).  1024 where the bundles of a level are no
// more than the compute units and have 128 tasks and more: then the time is one bundle's, most of it the chain of ranks
// (config 3's levels of up to 12 bundles 26 -> 19 us, the solve 773 -> 703 us, config 4's 1102 -> 1065; with fewer tasks
// 256 threads are faster, 11 against 13 us, and so they are with Move Specs, config 12's solve 3166 against 3220).
template <int T, bool LAY, bool MOVES>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(T == 512 ? 5 : 4))) void fill_kernel(
    const DevParams* __restrict__ P, const FillGeom g, const uint32_t* __restrict__ items, const uint32_t* __restrict__ starts,
    const ShapeRec* __restrict__ recs, const unsigned long long* __restrict__ masks, uint64_t* __restrict__ cost, uint16_t* __restrict__ arg,
    Counters* __restrict__ ctr) {
  extern __shared__ __align__(16) unsigned char smem[];
  FillLds L;
  carve_fill(smem, g, MOVES, L);
  const uint32_t tid = threadIdx.x, lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t i0 = starts ? starts[blockIdx.x] : blockIdx.x, n_it = starts ? starts[blockIdx.x + 1] - i0 : 1u;
  const uint32_t npass = P->npass, nops = P->nops, ndt = P->ndt, ndp = 1u << ndt, nwp = P->nwp, nw = ndp * nwp, log2V = P->log2V;
  const uint32_t nlay = g.nlay, psz = 1u << (2 * nops);
  constexpr uint32_t kXw = LAY && !MOVES ? 2u : 1u;      // Move-cost entries per (operand, source, destination)
  uint32_t n_rw = 0, ovf = 0;
  if (n_it > g.ni) { if (tid == 0) atomicOr(&ctr->overflow, 2u); return; }       // the work lists guarantee this cannot happen

  // ---- the items, one per lane of the first wave ----
  if (wave == 0) {
    uint32_t cnt = 0;
    if (lane < n_it) {
      const uint32_t item = items[i0 + lane];
      unsigned long long m[4] = {0, 0, 0, 0};
#pragma unroll
      for (int w = 0; w < 4; w++) if ((uint32_t)w < nw) m[w] = masks[(size_t)item * nw + w];
      const uint32_t si_i = item / npass, pass = item - si_i * npass;
      const ShapeRec R = recs[si_i];
      uint32_t si[4];
#pragma unroll
      for (int d = 0; d < 4; d++) si[d] = (R.si >> (8 * d)) & 0xFFu;
#pragma unroll
      for (int w = 0; w < 4; w++) { L.it_mask[lane * 4 + w] = m[w]; cnt += (uint32_t)__popcll(m[w]); }
      L.it_pass[lane] = pass; L.it_base[lane] = R.shape * P->G + (pass << log2V);
      L.it_si[lane] = R.si; L.it_nserial[lane] = R.n_serial; L.it_ntile[lane] = R.n_tile; L.it_mk[lane] = R.mk_var & 0xFFu;
      L.it_cnt[lane] = R.tile_cnt;
#pragma unroll
      for (int d = 0; d < 4; d++) L.it_lo[lane * 4 + d] = R.tile_lo[d];
#pragma unroll
      for (int i = 0; i < 5; i++) L.it_numel[lane * 5 + i] = R.numel[i];
      uint32_t rowM = 0, rowE = 0;
      uint64_t z = 0;
      if (P->kind == kKindF) {
        const uint32_t zc = pass == 0 ? P->zero[0] : pass == 1 ? P->zero[1] : pass == 2 ? P->zero[2] : P->zero[3];
        z = mul_or_limit(zc, R.numel[4]);
        if (P->chain) {
          // the table's k and n lists are this lattice's p list (and k and n lists)
          rowM = ((si[1] * P->nkM + si[2]) * P->nsz[3] + si[0]) * P->GM;
          rowE = ((si[1] * P->nkM + si[0]) * P->nsz[3] + si[3]) * P->GM;
        } else {
          rowM = ((si[1] * P->nkM + si[2] + P->kM_first) * P->nsz[3] + si[3]) * P->GM;
          rowE = (si[1] * P->nszE_n + si[3]) * P->GE;
        }
      } else if (P->split) {
        const uint32_t sh = si[1] * P->nsz[3] + si[3];
        rowM = sh * P->GM; rowE = sh * P->GE;
      }
      L.it_rowM[lane] = rowM; L.it_rowE[lane] = rowE; L.it_z[lane] = z;
      // (unpacked: widths at 2 * i, positions at 8 + 4 * i, their sum at 24)
      const uint32_t pv = R.mk_var >> 8;
      L.it_var[lane] = (pv & 0x3Fu) | (pv >> 6 & 7u) << 8 | (pv >> 9 & 7u) << 12 | (pv >> 12 & 7u) << 16 | (pv >> 15) << 24;
    }
    uint32_t incl = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(incl, d, 64);
      if ((int)lane >= d) incl += o;
    }
    if (lane < n_it) L.it_first[lane] = incl - cnt;
    if (lane == 63) L.it_first[n_it] = incl;
    if (lane < kMaxRanks + 2) L.rcnt[lane] = 0;
  }
  for (uint32_t i = tid; i < n_it * g.isz / 2; i += T) reinterpret_cast<uint32_t*>(L.idx)[i] = g.ns | g.ns << 16;
  if (tid < (1u << nlay)) L.t_cost[(MOVES ? g.cap : g.ns << nlay) + tid] = kInf;
  if (MOVES && tid == 0) L.tk0[g.ns] = (uint16_t)g.cap;
  __syncthreads();
  const uint32_t n_ent = L.it_first[n_it];
  if (n_ent > g.ns) { if (tid == 0) atomicOr(&ctr->overflow, 2u); return; }      // (nor this)

  // (what the next three steps read of the parameters does not depend on the items: it is requested
  // together with the first tile rewrites, so that one trip to memory serves all of them)
  auto tile_at = [&](uint32_t i, uint32_t e0, uint32_t& td) -> uint32_t {       // entry of the tile list behind LDS place i
    const uint32_t j = i / g.kt, e = e0 + (i - j * g.kt), cnts = L.it_cnt[j];
    uint32_t first = 0, q = ~0u;
    td = 0;
    if (e >= L.it_ntile[j]) return q;
#pragma unroll
    for (int d = 0; d < 4; d++) {
      const uint32_t cnt = P->tile_dim_ok[d] ? (cnts >> (8 * d)) & 0xFFu : 0u;
      if (e >= first && e < first + cnt) { td = d; q = L.it_lo[j * 4 + d] + (e - first); }
      first += cnt;
    }
    if (P->par) {        // the parallel loops over b, m, n follow
#pragma unroll
      for (int d = 0; d < 4; d++) {
        if (d == 2) continue;
        const uint32_t cnt = (cnts >> (8 * d)) & 0xFFu;
        if (e >= first && e < first + cnt) { td = 4 + d; q = L.it_lo[j * 4 + d] + (e - first); }
        first += cnt;
      }
    }
    return q;
  };
  auto put_tile = [&](uint32_t i, uint32_t td, const TileEntry& te) {           // first cell of the child's item, trips, id
    const uint32_t j = i / g.kt, si = L.it_si[j], d = td & 3u, sj = (si >> (8 * d)) & 0xFFu;
    const uint32_t stride = d == 0 ? P->shape_stride[0] : d == 1 ? P->shape_stride[1] : d == 2 ? P->shape_stride[2] : P->shape_stride[3];
    L.tl_cell[i] = L.it_base[j] - (sj - te.jt) * stride * P->G;                 // the serial table has the same geometry
    L.tl_trips[i] = td >= 4 ? (te.trips + P->threads - 1) / P->threads : te.trips;
    L.tl_id[i] = (td >= 4 ? P->par_base : P->tile_base) + d * P->maxs + te.jt;
  };
  uint32_t td0 = 0;
  const uint32_t q_tile0 = tid < n_it * g.kt ? tile_at(tid, 0, td0) : ~0u;
  const TileEntry te0 = P->tiles[q_tile0 == ~0u ? 0u : q_tile0];
  const uint32_t pos0 = (wave % nw % nwp) * 64u + lane, pe0 = P->pos_entry[pos0 < kMaxCombo ? pos0 : 0u];

  // ---- the admissible entries: by item, and counted by rank ----
  for (uint32_t jw = wave; jw < n_it * nw; jw += T / 64) {
    const uint32_t j = jw / nw, w = jw - j * nw, dt = w / nwp, pos = (w - dt * nwp) * 64u + lane;
    const unsigned long long m = L.it_mask[j * 4 + w];
    uint32_t slot = L.it_first[j];
#pragma unroll
    for (uint32_t u = 0; u < 3; u++) if (u < w) slot += (uint32_t)__popcll(L.it_mask[j * 4 + u]);
    if ((m >> lane) & 1ull) {
      slot += __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      const uint32_t pe = jw == wave ? pe0 : P->pos_entry[pos], pack = pe & 0xFFu, rank = (pe >> 8) & 0xFFu;       // pack | rank << 8 | mixed-radix index << 16
      L.ent[slot] = pack | dt << 8 | j << 10 | rank << 16 | (pe >> 16) << 20;
      L.idx[j * g.isz + dt * psz + pack] = (uint16_t)slot;
      L.place[slot] = (uint16_t)atomicAdd(&L.rcnt[rank], 1u);                       // its place among the rank's entries
    }
  }
  // Move costs: coefficient * elements per (converted, operand, source level - 1, destination level, transposed),
  // 0 = no such Move; of a Matmul whose Moves are Specs: what bind_kernel tabulated for the operand's size
  if (MOVES) {
    const uint32_t per_op = 6u << (2 * P->yb), per_size = P->bind_d * per_op;
    for (uint32_t i = tid; i < n_it * g.bt; i += T) {
      const uint32_t j = i / g.bt, r = i - j * g.bt, dc = r / (3u * per_op), q = r - dc * 3u * per_op, op = q / per_op;
      const uint32_t si = L.it_si[j], sm = (si >> 8) & 0xFFu, sk = (si >> 16) & 0xFFu, sn = si >> 24;
      const uint32_t rows = op == 1 ? sk : sm, cols = op == 0 ? sk : sn;
      L.bterm[i] = P->bind[((size_t)(op == 2 ? P->nszV * P->nszV : 0u) + rows * P->nszV + cols) * per_size + dc * per_op + (q - op * per_op)];
    }
  } else {
    for (uint32_t i = tid; i < n_it * g.bt; i += T) {
      const uint32_t j = i / g.bt, r = i - j * g.bt, x = kXw == 2 ? r & 1u : 0u, sd = (r / kXw) % 9u, co = (r / kXw) / 9u, cv = co / nops, op = co - cv * nops;
      const uint32_t src = sd / 3u + 1u, dst = sd - (src - 1u) * 3u;
      const uint32_t c = dst < src ? P->mcoef[op][src][dst][x] : 0u;
      L.bterm[i] = c ? mul_or_limit((uint64_t)c + (cv ? P->convert : 0u), L.it_numel[j * 5 + op]) : 0;
    }
  }
  if (q_tile0 != ~0u) put_tile(tid, td0, te0);
  auto stage_tiles = [&](uint32_t e0, uint32_t i0) {
    for (uint32_t i = i0; i < n_it * g.kt; i += T) {
      uint32_t td;
      const uint32_t q = tile_at(i, e0, td);
      if (q != ~0u) put_tile(i, td, P->tiles[q]);
    }
  };
  stage_tiles(0, tid + T);
  __syncthreads();

  // every wave keeps the ranks' first places in its lanes (lane r: rank r)
  uint32_t rank_first;
  {
    const uint32_t c = lane < P->nranks ? L.rcnt[lane] : 0u;
    uint32_t incl = c;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      const uint32_t o = __shfl_up(incl, d, 64);
      if ((int)lane >= d) incl += o;
    }
    rank_first = lane < P->nranks ? incl - c : n_ent;
  }
  // the entries in rank order (used after the tile phase)
  for (uint32_t s0 = 0; s0 < n_ent; s0 += T) {
    const uint32_t s = s0 + tid, en = L.ent[s < n_ent ? s : 0u];
    const uint32_t at = __shfl(rank_first, ent_rank(en), 64);
    if (s < n_ent) { const uint32_t k = at + L.place[s]; L.rl_ent[k] = en; L.rl_slot[k] = (uint16_t)s; }
  }
  // tasks: the entries' layouts
  uint32_t n_task;
  if (MOVES) {
    if (wave == 0) {
      uint32_t run = 0;
      for (uint32_t s0 = 0; s0 < n_ent; s0 += 64) {
        const uint32_t s = s0 + lane, c = s < n_ent ? 1u << (L.it_var[ent_item(L.ent[s])] >> 24) : 0u;
        uint32_t incl = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t o = __shfl_up(incl, d, 64);
          if ((int)lane >= d) incl += o;
        }
        if (s < n_ent) L.tk0[s] = (uint16_t)(run + incl - c);
        run += __shfl(incl, 63, 64);
      }
      if (lane == 0) L.rcnt[kMaxRanks + 1] = run;
    }
    __syncthreads();
    n_task = L.rcnt[kMaxRanks + 1];
    if (n_task > g.cap) { if (tid == 0) atomicOr(&ctr->overflow, 2u); return; }
    for (uint32_t s = tid; s < n_ent; s += T) {
      const uint32_t c = 1u << (L.it_var[ent_item(L.ent[s])] >> 24), t0 = L.tk0[s];
      for (uint32_t k = 0; k < c; k++) L.tslot[t0 + k] = (uint16_t)s;
    }
    __syncthreads();
  } else {
    n_task = n_ent << nlay;
  }

  // ---- 1. tile and bufferize candidates of every task (sub-Specs of other shapes / tables: final) ----
  uint32_t max_tile = 0;
  for (uint32_t j = 0; j < n_it; j++) { const uint32_t t = L.it_ntile[j]; max_tile = t > max_tile ? t : max_tile; }
  max_tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)max_tile);          // the same in every lane: kept as a scalar
  const bool has_buf = !MOVES && (P->kind == kKindF || P->split);
  const uint64_t s_serial = P->s, s_par = P->sync;
  const uint64_t* __restrict__ serial = P->costM;
  // few tasks: a quad of lanes per task, every fourth candidate each (fewer reads one after the other)
  const uint32_t lg = n_task * 4 <= T ? 2u : 0u, sub4 = lg ? tid & 3u : 0u;
  for (uint32_t e0 = 0; e0 == 0 || e0 < max_tile; e0 += g.kt) {
    if (e0) { __syncthreads(); stage_tiles(e0, tid); __syncthreads(); }
    for (uint32_t qb = 0; qb < n_task; qb += T >> lg) {
      const uint32_t q0 = qb + (tid >> lg);
      if (!lg && q0 >= n_task) break;
      const uint32_t q = q0 < n_task ? q0 : 0u;
      const uint32_t slot = MOVES ? (uint32_t)L.tslot[q] : q >> nlay, c = MOVES ? q - L.tk0[slot] : q & ((1u << nlay) - 1u);
      const uint32_t en = L.ent[slot], j = ent_item(en);
      const uint32_t v = variant_of<MOVES>(P, MOVES ? L.it_var[j] : 0u, c, ent_dt(en));
      const uint32_t off = ((ent_combo(en) * npass) << log2V) + v;
      const uint32_t all = L.it_ntile[j], n_here = all <= e0 ? 0u : all - e0 < g.kt ? all - e0 : g.kt;
      const uint32_t n_ser = L.it_nserial[j] > e0 ? L.it_nserial[j] - e0 : 0u;     // from here on parallel loops
      Eval e;
      e.best = kInf; e.arg = kNone; e.ovf = 0;
      if (e0 && sub4 == 0) { e.best = L.t_cost[q]; e.arg = L.t_arg[q]; }
      // trips * sub + s in 96 bits; reaching 2^62 = overflow.  A parallel loop's body is the
      // serial-only Spec (read from the serial table), its constant the synchronisation cost.
      for (uint32_t t0 = sub4; t0 < n_here; t0 += kBatch << lg) {
        uint64_t sub[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; u++) {
          const uint32_t t = t0 + (u << lg);
          sub[u] = kInf;
          if (t < n_here) sub[u] = (t >= n_ser ? serial : cost)[L.tl_cell[j * g.kt + t] + off];     // no request for a candidate that is not there
        }
#pragma unroll
        for (int u = 0; u < kBatch; u++) {
          const uint32_t t = t0 + (u << lg);
          if (t < n_here) {
            const bool fin = (uint32_t)(sub[u] >> 32) != ~0u;
            const uint32_t a = L.tl_trips[j * g.kt + t];
            const uint64_t lo = (uint64_t)a * (uint32_t)sub[u];
            const uint64_t hi = (uint64_t)a * (uint32_t)(sub[u] >> 32) + (lo >> 32);   // bits 32.. of the product
            const uint64_t cand = ((hi << 32) | (uint32_t)lo) + (t >= n_ser ? s_par : s_serial);
            const bool over = fin & (((hi >> 30) != 0) | (cand >= kLimit));
            e.ovf |= over ? 1u : 0u;
            const bool better = fin & !over & (cand < e.best);       // ids ascend, also over the stretches of kt tiles
            e.best = better ? cand : e.best;
            e.arg = better ? L.tl_id[j * g.kt + t] : e.arg;
          }
        }
      }
      if (has_buf && e0 + g.kt >= max_tile && sub4 == 0) {       // after the last tiles: its id is above theirs
        const uint32_t nb = task_bufferize(P, L.it_rowM[j], L.it_rowE[j], L.it_z[j], L.it_numel + j * 5, ent_pack(en), L.it_pass[j], v, e);
        if (q0 < n_task) n_rw += nb;
      }
      if (lg) { quad_min<0xB1>(e); quad_min<0x4E>(e); }
      if (q0 < n_task) {
        ovf |= e.ovf;
        if (sub4 == 0) {
          L.t_cost[q] = e.best; L.t_arg[q] = (uint16_t)e.arg;
          if (e0 == 0) n_rw += all;
        }
      }
    }
  }
  __syncthreads();

  // ---- 2. rank by rank: Moves, microkernels, the parked tile/bufferize candidate ----
  // Four lanes per task, one operand each (its Moves to every lower level and layout); the lanes'
  // candidates are then reduced to the lexicographic minimum of (cost, id).  All tables are indexed
  // directly; a level assignment that does not fit reads the tasks of entry ns (INF).  On levels
  // short of work (T = 256) the chain of ranks is what counts, and eight lanes per task halve a
  // lane's work in each: lane 4 * x + op takes the changes of layout x and x + 2.  Elsewhere it is
  // the instructions, most of which a lane spends whatever its number of candidates.
  constexpr uint32_t kTaskLanes = LAY && (T == 256 || T == 1024) ? 8u : 4u, kXLanes = kTaskLanes / 4u;
  const uint32_t op = tid & 3u, x = kXLanes == 2 ? (tid >> 2) & 1u : 0u;
  const uint32_t my_shift = op == 0 ? P->pack_shift[0] : op == 1 ? P->pack_shift[1] : op == 2 ? P->pack_shift[2] : P->pack_shift[3];
  const uint32_t my_lay = op == 0 ? P->lay_bit[0] : op == 1 ? P->lay_bit[1] : op == 2 ? P->lay_bit[2] : P->lay_bit[3];
  const uint32_t my_dt = op == 0 ? P->dt_bit[0] : op == 1 ? P->dt_bit[1] : op == 2 ? P->dt_bit[2] : P->dt_bit[3];
  const bool my_cv = (op == 0 ? P->can_convert[0] : op == 1 ? P->can_convert[1] : op == 2 ? P->can_convert[2] : P->can_convert[3]) != 0 && my_dt != kNoBit;
  const uint32_t base_bf = op == 0 ? P->base_bf16[0] : op == 1 ? P->base_bf16[1] : op == 2 ? P->base_bf16[2] : P->base_bf16[3];
  const uint32_t my_lw = op == 0 ? P->lay_w[0] : op == 1 ? P->lay_w[1] : op == 2 ? P->lay_w[2] : P->lay_w[3];
  const bool my_part = op < nops && (x == 0 || my_lay != kNoBit);
  const uint32_t xw = MOVES ? P->xw : 2u, id0 = P->move_base + op * (P->NL - 1u) * xw * 2u + x * 2u;
  const uint32_t yb = MOVES ? P->yb : 0u, nranks = P->nranks, bind_d = MOVES ? P->bind_d : 1u;
  const uint32_t my_fb = my_lay != kNoBit ? my_lay - ndt : 0u, op_row = op * 9u * kXw + x;
  // (with packed layouts the entries of a rank may have different numbers of tasks: lanes for the most of any item)
  uint32_t lays = nlay;
  if (MOVES) {
    lays = 0;
    for (uint32_t j = 0; j < n_it; j++) { const uint32_t w = L.it_var[j] >> 24; lays = w > lays ? w : lays; }
  }
  for (uint32_t r = 0; r < nranks; r++) {
    const uint32_t r0 = lane_of(rank_first, r), r1 = lane_of(rank_first, r + 1);
    if (r0 == r1) continue;
    const uint32_t n_here = (r1 - r0) << lays;
    for (uint32_t qb = 0; qb < n_here; qb += T / kTaskLanes) {
      const uint32_t qq = qb + tid / kTaskLanes;
      bool active = qq < n_here;
      const uint32_t k = r0 + (active ? qq >> lays : 0u);
      const uint32_t slot = L.rl_slot[k], en = L.rl_ent[k], j = ent_item(en), pack = ent_pack(en), dt = ent_dt(en);
      uint32_t c = active ? qq & ((1u << lays) - 1u) : 0u, var = 0;
      if (MOVES) {
        var = L.it_var[j];
        active = active && c < (1u << (var >> 24));
        c = active ? c : 0u;
      }
      const uint32_t q = MOVES ? L.tk0[slot] + c : (slot << nlay) + c;
      Eval parked;
      parked.best = L.t_cost[q]; parked.arg = L.t_arg[q];
      const uint32_t mk_shape = L.it_mk[j];
      Eval e;
      e.best = kInf; e.arg = kNone;
      uint32_t hi_or = 0;           // OR of the high words of all finite Move candidates
      const uint32_t src = (pack >> my_shift) & 3u;
      const bool on = active && my_part && src != 0;
      if (__any(on)) {
        const uint32_t src1 = on ? src - 1u : 0u, at = j * g.isz + pack;
        const uint32_t bf = my_dt != kNoBit ? (dt >> my_dt) & 1u : base_bf;
        for (uint32_t cv = 0; cv < ndp && cv < 2u; cv++) {             // as it is, then converted
          const bool plane = on && (cv == 0 || (my_cv && bf));
          if (cv && !__any(plane)) break;
          const uint32_t dt2 = cv ? dt & ~(1u << (my_dt & 31u)) : dt;
          uint32_t to[3];
#pragma unroll
          for (uint32_t dst = 0; dst < 3; dst++) to[dst] = L.idx[at + dt2 * psz - (plane && dst < src ? (src - dst) << my_shift : 0u)];
          if (MOVES) {
            // my operand's field inside c, its width
            const uint32_t fw = (var >> (2 * op)) & 3u, fb = (var >> (8 + 4 * op)) & 7u, y0 = (c >> fb) & ((1u << fw) - 1u);
            const uint32_t row = j * g.bt + ((((bind_d == 3 && bf ? 1u + cv : 0u) * 3u + op) * 6u + (src1 + 1u) * src1 / 2u) << (2 * yb)) + (y0 << yb);
            for (uint32_t xx = x; xx < xw; xx += kXLanes) {
              const bool counts = plane && xx < (1u << my_lw);
              const bool exists = counts && xx < (1u << fw);          // (a packed layout that this size cannot have: no such Spec)
              n_rw += counts ? src : 0u;
              if (!__any(exists)) continue;
#pragma unroll
              for (uint32_t dst = 0; dst < 3; dst++) {
                const bool ok = exists && dst < src;
                const uint64_t b = L.bterm[ok ? row + (dst << (2 * yb)) + (y0 ^ xx) : 0u], t = L.t_cost[ok ? L.tk0[to[dst]] + (c ^ (xx << fb)) : q];
                const bool fin = ok && (uint32_t)(b >> 32) != ~0u && (uint32_t)(t >> 32) != ~0u;
                const uint64_t cand = t + b;                          // each at most 2^62 when finite: no wrap
                hi_or |= fin ? (uint32_t)(cand >> 32) : 0u;
                consider(e, cand, id0 + (dst * xw + (xx - x)) * 2u + cv, fin);
              }
            }
          } else {
            const uint32_t row = j * g.bt + cv * nops * 9u * kXw + op_row + src1 * 3u * kXw;
            constexpr uint32_t kMine = kXw / kXLanes ? kXw / kXLanes : 1u;      // changes of layout per lane
            uint64_t b[3][kMine], t[3][kMine];
#pragma unroll
            for (uint32_t dst = 0; dst < 3; dst++)
#pragma unroll
              for (uint32_t u = 0; u < kMine; u++) {
                b[dst][u] = L.bterm[row + dst * kXw + u];
                t[dst][u] = L.t_cost[(to[dst] << nlay) + (c ^ ((x + u) << my_fb))];
              }
#pragma unroll
            for (uint32_t dst = 0; dst < 3; dst++)
#pragma unroll
              for (uint32_t u = 0; u < kMine; u++) {
                const bool counts = plane && b[dst][u] != 0;          // 0 = no such Move (and no destination at or above src)
                n_rw += counts ? 1u : 0u;
                const bool fin = counts && (uint32_t)(t[dst][u] >> 32) != ~0u;
                const uint64_t cand = t[dst][u] + b[dst][u];          // t < 2^62 when finite, b <= 2^62: no wrap
                hi_or |= fin ? (uint32_t)(cand >> 32) : 0u;
                const uint32_t id = id0 + dst * 4u + u * 2u + cv;
                if (cv) consider(e, cand, id, fin);
                else {
                  const bool better = fin && cand < e.best;           // ids ascend
                  e.best = better ? cand : e.best;
                  e.arg = better ? id : e.arg;
                }
              }
          }
        }
      }
      if (hi_or >> 30) ovf |= 1u;   // bit 62 of some finite candidate: the solve reports overflow
      quad_min<0xB1>(e);            // lanes ^ 1
      quad_min<0x4E>(e);            // lanes ^ 2
      if (kXLanes == 2) quad_min<0x141>(e);  // the other quad of eight (mirrored: the lanes of a quad agree by now)
      if (active && (tid & (kTaskLanes - 1u)) == 0) {
        // the task's first lane adds the microkernels (lowest ids) and the parked candidate (highest), and stores
        consider(e, parked.best, parked.arg);
        if (mk_shape) {
          const uint32_t v = variant_of<MOVES>(P, var, c, dt), si = L.it_si[j];
          for (uint32_t mm = P->mk_entry[(pack << log2V) + v] & mk_shape; mm; mm &= mm - 1) {
            const uint32_t m = (uint32_t)__ffs((int)mm) - 1u;
            Shape S;
#pragma unroll
            for (int d = 0; d < 4; d++) S.d[d] = P->sizes[d][(si >> (8 * d)) & 0xFFu];
            const uint64_t ck = mul_or_limit(P->mk_cost[m], mk_shape_reps(P, S, m));
            if (ck >= kLimit) ovf |= 1u; else consider(e, ck, m);
            n_rw++;
          }
        }
        L.t_cost[q] = e.best;
        L.t_arg[q] = (uint16_t)e.arg;
      }
    }
    __syncthreads();
  }
  // ---- 3. results to the table, a task per lane: inside the rank loop every chunk would wait for
  // the previous chunk's stores (stores count on the same counter as loads here) ----
  for (uint32_t q = tid; q < n_task; q += T) {
    const uint32_t slot = MOVES ? (uint32_t)L.tslot[q] : q >> nlay, c = MOVES ? q - L.tk0[slot] : q & ((1u << nlay) - 1u);
    const uint32_t en = L.ent[slot], j = ent_item(en);
    const uint32_t cell = L.it_base[j] + ((ent_combo(en) * npass) << log2V) + variant_of<MOVES>(P, MOVES ? L.it_var[j] : 0u, c, ent_dt(en));
    cost[cell] = L.t_cost[q];
    arg[cell] = L.t_arg[q];
  }
  flush_counters(ctr, n_rw, ovf);
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
__global__ __launch_bounds__(256) void fill_ones_short_kernel(uint4* __restrict__ p, size_t n16) {
  const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u);
  const size_t i0 = (size_t)blockIdx.x * 1024u + threadIdx.x;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const size_t i = i0 + (size_t)k * 256u;
    if (i < n16) p[i] = ones;
  }
}

void launch_fill_ones(void* p, size_t bytes, hipStream_t stream, bool short_lived) {
  const size_t n16 = bytes / 16;
  if (n16 && short_lived) {
    size_t done = 0;
    while (done < n16) {          // (grids stay below 2^31 workgroups)
      const size_t part = n16 - done < ((size_t)1 << 40) ? n16 - done : ((size_t)1 << 40);
      hipLaunchKernelGGL(fill_ones_short_kernel, dim3((uint32_t)((part + 1023) / 1024)), dim3(256), 0, stream, (uint4*)p + done, part);
      done += part;
    }
  } else if (n16) {
    const size_t blocks = (n16 + 255) / 256;
    hipLaunchKernelGGL(fill_ones_kernel, dim3((uint32_t)(blocks < 16384 ? blocks : 16384)), dim3(256), 0, stream,
                       (uint4*)p, n16);
  }
  if (bytes % 16) (void)hipMemsetAsync((char*)p + n16 * 16, 0xFF, bytes % 16, stream);
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
    const uint32_t pack = P->pos_info[c0 + ci] & 0xFFu;
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
    const uint32_t pack = P->pos_info[c0 + ci] & 0xFFu;
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
// Items of at most this many tasks go into bundles: everything where a whole shape is that small.
uint32_t fill_small_max(uint32_t max_task) { return max_task <= 512 ? max_task : 256; }

// Items per bundle at most (the tables of Move costs of packed layouts are large).
static uint32_t fill_items(const DevParams& P) { return P.moves ? 4u : 8u; }

static FillGeom fill_geom(const DevParams& P, uint32_t max_task, bool wide) {
  FillGeom g;
  g.ni = wide ? 1u : fill_items(P);
  g.cap = wide ? max_task : kBundle + fill_small_max(max_task);
  g.kt = wide ? 64u : 24u;
  g.bt = P.moves ? P.bind_d * 3u * (6u << (2 * P.yb)) : (P.ndt ? 2u : 1u) * P.nops * (P.nlay ? 18u : 9u);
  g.isz = (1u << P.ndt) << (2 * P.nops);
  g.nlay = P.nlay;
  const uint32_t entries = (P.ncombo << P.ndt) * g.ni;
  g.ns = P.moves ? (g.cap < entries ? g.cap : entries) : g.cap >> P.nlay;
  return g;
}

// Workgroups of the sort kernels: the levels' tiles.
static uint32_t sort_tiles(const uint32_t* level_off, uint32_t n_levels, uint32_t npass) {
  uint32_t n = 0;
  for (uint32_t l = 0; l < n_levels; l++) n += ((level_off[l + 1] - level_off[l]) * npass + kSortTile - 1) / kSortTile;
  return n;
}
// A level's weights are added up in 32 bits (an item weighs at least kBundle / fill_items; the
// tasks themselves are fewer than 2^32), and a launch has fewer than 2^32 threads: the plan's has
// four per shape, a level's 128 per bundle.
bool plan_fits(const DevParams& h, uint32_t n_shapes, const uint32_t* level_off, uint32_t n_levels) {
  if (n_shapes >= (1u << 30) - 4 * kPlanShapes) return false;
  for (uint32_t l = 0; l < n_levels; l++)
    if ((uint64_t)(level_off[l + 1] - level_off[l]) * h.npass >= (1ull << 32) / (kBundle / fill_items(h))) return false;
  return true;
}
size_t plan_bytes_recs(uint32_t n_shapes) { return (size_t)n_shapes * sizeof(ShapeRec); }
size_t plan_bytes_sort(const uint32_t* level_off, uint32_t n_levels, uint32_t npass) { return (size_t)sort_tiles(level_off, n_levels, npass) * 32 + 16; }

void launch_plan(const DevParams* P, const DevParams& h, uint32_t n_shapes, uint32_t max_task, const uint32_t* level_shapes,
                 const uint32_t* level_off, const uint32_t* h_level_off, uint32_t n_levels, const PlanBuffers& B, uint32_t* fitmap, Counters* ctr,
                 void* prefill_cost, void* prefill_arg, hipStream_t stream) {
  const uint32_t per_wave = plan_shapes(n_shapes);
  hipLaunchKernelGGL(plan_kernel, dim3((n_shapes + 4 * per_wave - 1) / (4 * per_wave)), dim3(256), 0, stream, P,
                     n_shapes, per_wave, fit_map_stored(h) ? 1u : 0u, level_shapes, (ShapeRec*)B.recs, B.masks, B.item_tasks, fitmap, ctr, (uint4*)prefill_cost, (uint4*)prefill_arg);
  const uint32_t tiles = sort_tiles(h_level_off, n_levels, h.npass), small_max = fill_small_max(max_task), min_weight = kBundle / fill_items(h);
  uint4* parts = (uint4*)B.sort_tmp;
  uint32_t* sums = tiles > n_levels ? (uint32_t*)(parts + tiles) : nullptr;
  if (sums) {
    hipLaunchKernelGGL(sort_sums_kernel, dim3(tiles), dim3(kSortThreads), 0, stream, level_off, h.npass, B.item_tasks, small_max, sums);
    hipLaunchKernelGGL(sort_work_kernel, dim3(tiles), dim3(kSortThreads), 0, stream, level_off, n_levels, h.npass, B.item_tasks, small_max,
                       min_weight, 0u, sums, parts, B.list_small, B.bundle_first, B.list_wide, B.list_cnt);
  }
  hipLaunchKernelGGL(sort_work_kernel, dim3(tiles), dim3(kSortThreads), 0, stream, level_off, n_levels, h.npass, B.item_tasks, small_max,
                     min_weight, 1u, sums, parts, B.list_small, B.bundle_first, B.list_wide, B.list_cnt);
}

void launch_bind(const DevParams* P, uint64_t* bind, uint32_t n, hipStream_t stream) {
  hipLaunchKernelGGL(bind_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, P, bind, n);
}

template <int T>
static void launch_items(const DevParams* P, const DevParams& h, const FillGeom& g, uint32_t n, const uint32_t* items, const uint32_t* starts,
                         const PlanBuffers& B, uint64_t* cost, uint16_t* arg, Counters* ctr, hipStream_t stream) {
  FillLds L;
  const uint32_t lds = carve_fill(nullptr, g, h.moves != 0, L);
  const ShapeRec* recs = (const ShapeRec*)B.recs;
  if (h.moves) {
    if constexpr (T < 1024)       // (more threads are slower with Move Specs, and never asked for: below)
      hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_kernel<T, true, true>), dim3(n), dim3(T), lds, stream, P, g, items, starts, recs, B.masks, cost, arg, ctr);
  } else if (h.nlay) {
    hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_kernel<T, true, false>), dim3(n), dim3(T), lds, stream, P, g, items, starts, recs, B.masks, cost, arg, ctr);
  } else {
    hipLaunchKernelGGL(HIP_KERNEL_NAME(fill_kernel<T, false, false>), dim3(n), dim3(T), lds, stream, P, g, items, starts, recs, B.masks, cost, arg, ctr);
  }
}

// The bundles of one dependency level (starts = nullptr: every item is a bundle of its own).
void launch_fill_level(const DevParams* P, const DevParams& h, uint32_t max_task, uint32_t n, const uint32_t* items, const uint32_t* starts,
                       uint32_t lg_tasks, const PlanBuffers& B, uint64_t* cost, uint16_t* arg, Counters* ctr, hipStream_t stream) {
  if (!n) return;
  const FillGeom g = fill_geom(h, max_task, false);
  if (n >= kMinBundles) launch_items<128>(P, h, g, n, items, starts, B, cost, arg, ctr, stream);
  else if (n <= kFewBundles && lg_tasks >= kManyTasks && !h.moves) launch_items<1024>(P, h, g, n, items, starts, B, cost, arg, ctr, stream);
  else launch_items<256>(P, h, g, n, items, starts, B, cost, arg, ctr, stream);
}
// Its wide items.
void launch_fill_wide(const DevParams* P, const DevParams& h, uint32_t max_task, uint32_t n, const uint32_t* items, const PlanBuffers& B,
                      uint64_t* cost, uint16_t* arg, Counters* ctr, hipStream_t stream) {
  if (n) launch_items<512>(P, h, fill_geom(h, max_task, true), n, items, nullptr, B, cost, arg, ctr, stream);
}

}  // namespace mrl
