// Internal: host-side launchers of the kernels in fill.hip and compress.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <tuple>
#include "dev_params.h"

namespace mrl {

// A launch that gives its own status.  (The runtime's last error may be one that another call of the
// calling thread left there: it says nothing about this launch.)
template <class... P, class... A>
hipError_t launch_checked(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t st, const A&... args) {
  std::tuple<P...> v(args...);
  return std::apply([&](P&... a) {
    void* at[] = {(void*)&a...};
    return hipLaunchKernel((const void*)kernel, grid, block, at, 0, st);
  }, v);
}

// The place of set bit number i of a word.
__device__ __forceinline__ uint32_t nth_bit(unsigned long long x, uint32_t i) {
  uint32_t at = 0;
#pragma unroll
  for (uint32_t d = 32; d > 0; d >>= 1) {
    const uint32_t n = (uint32_t)__popcll(x >> at & ((1ull << d) - 1ull));
    if (i >= n) { i -= n; at += d; }
  }
  return at;
}

// Table geometry passed by value to the compression kernels (cells < 2^32).
struct Geo {
  uint32_t ndim, n;
  uint32_t ext[16], stride[16];
};

// Device buffers of the work lists.
struct PlanBuffers {
  void* recs;                              // plan_bytes_recs
  unsigned long long* masks;
  const uint32_t *level_shapes, *level_off, *blk_off;       // shapes by dependency level; first shape and first block (unit_blocks) of every level
  uint32_t *cnt, *seg;                     // [ranks][blocks], [levels][ranks]
  uint32_t* host_diag;                     // pinned host memory: the diagonals' first places in the list, and the end
  void* list;                              // 8 bytes per unit
};
size_t plan_bytes_recs(uint32_t n_shapes);
// Blocks of items that the work lists are made in; blk_off (may be null): first block of every level, and their number.
uint32_t unit_blocks(const uint32_t* level_off, uint32_t n_levels, uint32_t npass, uint32_t* blk_off);
// Whether the work lists can hold the lattice's dependency levels.  h: the host's copy of *P.
bool plan_fits(const DevParams& h, uint32_t n_shapes, const uint32_t* level_off, uint32_t n_levels);
// h: the host's copy of *P.
void launch_plan(const DevParams* P, const DevParams& h, uint32_t n_levels, uint32_t n_blk, const PlanBuffers& B, Counters* ctr, hipStream_t stream);
// Behind the plan: which cells fit, in table order, n_words words and two of zeros.
void launch_fit_map(const DevParams* P, uint32_t n_specs, const PlanBuffers& B, uint32_t* fitmap, uint32_t n_words, hipStream_t stream);
// Units [w0, w0 + w_len) of the work list, which lie on diagonals d0 to d1, to its place; none if there are none_from units and more.
// h_blk_off: the host's copy of the first block of every level.
void launch_list_units(const DevParams* P, const DevParams& h, uint32_t n_levels, const uint32_t* h_blk_off, const PlanBuffers& B, uint32_t w0, uint32_t w_len, uint32_t d0, uint32_t d1,
                       uint64_t none_from, hipStream_t stream);
// The costs of the alloc-bindings of a Matmul whose Moves are Move Specs, from its Move table.
void launch_bind(const DevParams* P, uint64_t* bind, uint32_t n, hipStream_t stream);
// What the kernels of the diagonals read of the parameters, by value: they are short, and every read of the
// parameters in device memory would be another round trip.
struct FillArgs {
  const DevParams* P;
  const void* recs;
  const TileStep* steps;
  uint64_t* cost;
  uint16_t* arg;
  Counters* ctr;
  const uint64_t *costM, *costE;
  const uint8_t* mk_entry;
  uint32_t nops, NL, G, log2V, ndt, unit_lay;
  uint32_t mstride[4], pack_shift[4], lay_bit[4];
  uint32_t lay_xor[4], cv_bit[4];                              // layout bit of an operand's entry, dtype bit that a converting Move clears (0: none)
  uint32_t convert, s, sync, move_base, buf_id, par_shift;
  uint32_t nranks, npass, nwp;
  uint32_t lg_split;                                           // lanes that share an entry where it is split: 1 << lg_split
  uint32_t has_buf, split, chain, GM, VM, GE, VE, nszE_n, kM_first, nkM, nsz3, layM[3], layE[3], zero[4];
};
FillArgs fill_args(const DevParams* d_P, const DevParams& h, const PlanBuffers& B, uint64_t* cost, uint16_t* arg, Counters* ctr);
// Diagonals that one launch takes: n of them, diagonal i at places [start[i], start[i + 1]) of the list.  Small ones
// (small_diagonal) go into a chain, any other is a launch of its own.
constexpr uint32_t kRunMost = 63, kChainThreads = 1024, kSplitTasks = 32768, kBareSplitTasks = 131072;
struct DiagRun { uint32_t n, chain, start[kRunMost + 1]; };
uint64_t by_shapes_from(const DevParams& h, uint32_t n_shapes, uint32_t n_levels);      // units
uint32_t units_for_a_launch(const DevParams& h);
void launch_fill_shapes(const FillArgs& A, const DevParams& h, const unsigned long long* masks, uint32_t first, uint32_t n, hipStream_t stream);
bool small_diagonal(const FillArgs& A, uint32_t n_units);
uint32_t most_units(const FillArgs& A);            // that one launch takes
void launch_fill_diagonals(const FillArgs& A, const DevParams& h, const void* list, const DiagRun& run, hipStream_t stream);

// Segments of one launch of the bounded fill: segment i is (dependency level of shapes, rank)
// = shapes [first_shape, first_shape + n_shapes) of the level-ordered shape list at rank[i], and
// owns workgroups [block0[i], block0[i + 1]).  Where a wave takes a stretch of one (shape, level
// assignment) (fill_by_units): lanes_per_wave entries of it, waves_per_unit waves for all of them.
constexpr uint32_t kBoundSegs = 32;
struct BoundSegs {
  uint32_t n, waves_per_unit, lanes_per_wave;
  uint32_t first_shape[kBoundSegs], n_shapes[kBoundSegs], rank[kBoundSegs], block0[kBoundSegs + 1];
};
// mode 0: a lattice with memory bounds; 1: Move Specs.
// qv: entries per level assignment.
bool fill_by_units(int mode, uint64_t qv);
void launch_fill_bounded(const DevParams* P, int mode, bool units, const uint32_t* all_level_shapes, const BoundSegs& segs, uint64_t* cost,
                         uint16_t* arg, Counters* ctr, hipStream_t stream);
void launch_fill_ones(void* p, size_t bytes, hipStream_t stream);
void launch_prefill(uint64_t* cost, uint16_t* arg, size_t n, hipStream_t stream);
void launch_zero_words(unsigned long long* p, uint32_t n, hipStream_t st);
void launch_head_flags(const Geo& g, uint32_t a0, const uint64_t* cost, const uint16_t* arg, const uint32_t* fitmap,
                       const uint32_t* axis_sizes,
                       unsigned long long* maskD, unsigned long long* maskC, unsigned long long* lineD,
                       unsigned long long* lineC, hipStream_t st);
void scan_mask_words(const unsigned long long* mask, uint32_t n_words, uint32_t* tile_tmp, uint32_t* prefix,
                     uint32_t* total, hipStream_t st);
void scan_flags(const uint8_t* flags, uint32_t n, uint32_t* tile_tmp, uint32_t* pos, uint32_t* total, hipStream_t st);
// Live boxes (alive[b]) move to dense arrays: box b becomes box pos[b].
void launch_compact_boxes(uint32_t n, const uint8_t* alive, const uint32_t* pos, const uint32_t* bcell, const void* blen,
                          uint32_t* cell2, void* len2, uint8_t* alive2, hipStream_t st);
// The first generic pass (axis a1) done on the cells, for tables whose a0 and a1 have strides of
// whole mask words with a1 outside a0 and at most 64 steps on a1: runs = the mask of pass 0,
// mask2 = runs without the heads that this pass folds into the run before them on a1, col = one
// word per column of cells along a1 (zero before), bit c set where the run at step c was folded.
void launch_second_axis(const Geo& g, uint32_t a0, uint32_t a1, bool is_cost, const unsigned long long* runs,
                        const unsigned long long* line, const uint32_t* fitmap, const uint64_t* cost, const uint16_t* arg,
                        const uint32_t* axis_sizes, unsigned long long* mask2, unsigned long long* col, hipStream_t st);
// col != nullptr: mask is launch_second_axis's mask2 and every box gets its chain's length on a1.
void launch_make_boxes(const Geo& g, uint32_t a0, const unsigned long long* mask, const uint32_t* prefix,
                       const unsigned long long* line, const unsigned long long* col, uint32_t a1, uint32_t* bcell,
                       void* blen, uint8_t* alive, hipStream_t st);
// One merge pass along axis a.  After a compaction the mask still ranks boxes by their old index:
// old_alive / remap (the compaction's alive and pos) translate it; nullptr before.
void launch_axis_pass(const Geo& g, uint32_t a, uint8_t stamp, bool is_cost, uint32_t n_boxes, const uint8_t* old_alive,
                      const uint32_t* remap, const uint32_t* bcell, void* blen, uint8_t* alive, uint32_t* next,
                      uint32_t* block_linked, const unsigned long long* mask, const uint32_t* prefix, const uint64_t* cost,
                      const uint16_t* arg, const uint32_t* axis_sizes, hipStream_t st);
// The trailing passes over axes of extent 2 whose stride is at most 32 cells, in pass order.
struct TailAxes {
  uint32_t n;
  uint32_t axis[8], stride[8];
};
void launch_tail_pairs(const TailAxes& T, bool is_cost, uint32_t n_words, const unsigned long long* mask,
                       const uint32_t* prefix, const uint8_t* old_alive, const uint32_t* remap, void* blen, uint8_t* alive,
                       const uint64_t* cost, const uint16_t* arg, hipStream_t st);
void launch_emit(const Geo& g, const DevParams* P, bool is_cost, uint32_t n_boxes, const uint32_t* bcell,
                 const void* blen,
                 const uint8_t* alive, const uint32_t* pos, const uint64_t* cost, const uint16_t* arg, uint32_t* fcell,
                 void* flen, uint64_t* fv0, uint64_t* fv1, hipStream_t st);
// n boxes of a final list as the 80-byte records of the interface; out: pinned host memory, 16-byte aligned.
hipError_t launch_expand_boxes(const Geo& g, uint32_t n, const uint32_t* fcell, const void* flen, const uint64_t* fv0, const uint64_t* fv1, void* out,
                         hipStream_t st);
// idx, cost_out, arg_out: device memory or pinned host memory.
hipError_t launch_gather(const uint64_t* idx, uint32_t n, const uint64_t* cost, const uint16_t* arg, uint64_t* cost_out,
                   uint16_t* arg_out, hipStream_t st);

// The entries of a Spec, of the Spec its rewrite leads to, and so on.
struct ChainEntry { uint64_t cost; uint32_t cell, arg; };
constexpr uint32_t kChainMost = 64;
struct ChainWalk {
  Geo g;
  uint32_t cell, x[16];                     // where the walk starts: linear index, coordinate
  uint32_t move_base, tile_base, buf_id, maxs, xw, n_dst;      // rewrite ids (mrl_rewrite_decode)
  uint32_t moves, tiles;                    // 1: go on through Moves / tile loops
  int lay_axis[5], dt_axis[5];              // coordinate axes of an operand's layout and data type, -1 if none
};
// At most kChainMost entries to out, their number (at least 1) to n_out: device or pinned host memory.
hipError_t launch_chain(const ChainWalk& w, const uint64_t* cost, const uint16_t* arg, ChainEntry* out, uint32_t* n_out, hipStream_t st);

// Point lookups in a final box list: a packed hierarchy of bounding boxes over the list's order.
constexpr uint32_t kIndexFan = 8;          // children per node
constexpr uint32_t kIndexMaxLevels = 12;   // 8^11 > 2^32 boxes
struct alignas(32) BoxBounds { uint8_t lo[16], hi[16]; };   // inclusive corners, one byte per axis
struct IndexLevels {
  uint32_t n_levels;                       // level 0 = the boxes; the top level has at most kIndexFan nodes
  uint32_t count[kIndexMaxLevels], off[kIndexMaxLevels];    // nodes per level, first node of the level
  uint32_t total;
};
IndexLevels index_levels(uint32_t n_boxes);
void launch_build_index(const Geo& g, const IndexLevels& L, const uint32_t* fcell, const void* flen, BoxBounds* nodes,
                        hipStream_t st);
// One of the two final lists with its index.
struct LookupList {
  IndexLevels L;
  const BoxBounds* nodes;
  const uint32_t* fcell;
  const uint64_t *fv0, *fv1;
};
// lists: decisions, costs.  points: 16 bytes per point (coordinates, zero padded); vols: the volume
// b*m*k*n of each.  miss: a byte per list and point (n_points apart), 1 where no box holds the point.
hipError_t launch_lookup(const Geo& g, const LookupList lists[2], const void* points, const uint64_t* vols, uint32_t n_points,
                   uint64_t* cost_out, uint16_t* arg_out, uint8_t* miss, hipStream_t st);

// ---- the merge word by word (rowmerge.hip), for tables whose shapes are whole mask words
constexpr uint32_t kRowLevels = 5;         // level axes at most
constexpr uint32_t kRowInfoBytes = 64;
constexpr uint32_t kRowShapeWords = 256;   // words of a shape at most
// The size axes n, k, m, b, or k, m, b, n where there is one size along n (it then is the axis called b here, of one step; an
// axis of one step is never merged along, so that the order is the same), and so on; inside a shape the level axes, four values each (level axis i, in merge order, is the bits
// [lv + 2 i, lv + 2 i + 2) of a cell's place), then those of layouts and dtypes (fields of the lv bits below).
struct RowGeo {
  uint32_t en, ek, em, eb;                 // en: at most 64
  uint32_t axis[4];                        // the coordinate axes that b, m, k, n are here
  uint32_t G, nw, lg_nw;                   // cells and 64-cell words of a shape
  uint32_t n_shapes, n_planes;             // planes: (b, m, word of the shape)
  uint32_t lv, n_levels, n_inner, level_axis;      // n_inner: axes inside a shape, n_levels and a field each; level_axis: coordinate axis of level axis 0 (the others lie before it)
  uint32_t var_first, var_two, ndt;        // bits at which a layout or dtype field starts; which are two bits wide; dtype bits (the lowest, merged last)
  uint32_t var_axis[6];                    // coordinate axis of the field that starts at a bit
};
enum : uint32_t { kLongTotal = 0, kHeadsTotal = 1, kRowsTotal = 2, kBoxesTotal = 3, kBoxesFirst = 4, kRowTotals = 5 };     // (the first two are written as one)
struct RowBufs {
  uint32_t *rows, *first;                  // per plane: rows kept, index of its first
  void* info;                              // per kept row: kRowInfoBytes
  uint32_t *cnt, *start;                   // per list and shape: boxes, boxes before
  void* sum;                               // rows_sum_bytes
  uint32_t *tot;                           // kRowTotals
  char* dyn;                               // what depends on the contents: word arrays, extents, final lists
  uint64_t room;                           // bytes there
};
size_t rows_sum_bytes(const RowGeo& g);
// The whole merge and the final lists; nothing is read back.  sizes: DevParams::sizes on the device.
void launch_rows(const RowGeo& g, const RowBufs& B, const uint64_t* cost, const uint16_t* arg, const uint32_t* fitmap,
                 const uint32_t* sizes, hipStream_t st);
// Whether the words of so many kept rows fit room bytes (a plane keeps one row at least, ek at most).
bool row_words_fit(const RowGeo& g, uint64_t n_rows, uint64_t room);
// Whether all of it fits room bytes whatever the table holds.
bool rows_always_fit(const RowGeo& g, uint64_t room);
// Adds the number of rows that will be kept to *total, from the fit map alone.
void launch_row_total(const RowGeo& g, const uint32_t* fitmap, uint32_t* total, hipStream_t st);
// Given the totals: whether all of it fitted (nothing valid was written if not), where in dyn the lists lie, and the end.
bool rows_fit(const RowGeo& g, const uint32_t* tot, uint64_t room, uint64_t list_at[2], uint64_t* end);

constexpr uint32_t kScanTileItems = 2048;   // items per scan tile (tile_tmp needs n/2048 + 1 words)

}  // namespace mrl
