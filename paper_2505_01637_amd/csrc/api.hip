// C ABI of the library (include/morello_mi355x.h) and the host side of the
// solver: descriptor validation, coordinate system (Section 4.1), dependency
// levels of the bottom-up fill (Section 4 run in reverse), launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <condition_variable>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "../../include/morello_mi355x.h"
#include "compress.h"
#include "dev_params.h"

using namespace mrl;

static thread_local char g_err[512] = "";

static int32_t fail(int32_t code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
  return code;
}

#define HIP_TRY(expr)                                                                              \
  do {                                                                                             \
    hipError_t e_ = (expr);                                                                        \
    if (e_ != hipSuccess) return fail(MRL_E_HIP, "%s: %s", #expr, hipGetErrorString(e_));          \
  } while (0)

struct mrl_target {
  mrl_target_desc d;
};

namespace {

constexpr size_t kAlign = 256;
constexpr uint32_t kEmitChunk = 16384;     // boxes per launch of mrl_emit_compressed
constexpr uint32_t kQueryChunk = 32768;    // Specs per launch of a query in the dense table
#ifndef MRL_SECOND_ON_CELLS
#define MRL_SECOND_ON_CELLS 1
#endif
constexpr bool kSecondOnCells = MRL_SECOND_ON_CELLS;
constexpr uint64_t kStretch = 8;            // a wave of fill_units_kernel takes at most this many times 64 entries, and
constexpr uint64_t kFullWaves = 4096;       // more than one only where this many waves are left: its candidates' constants
                                            // cost a wave as much as two steps do (config 7's fill: stretch 4 and 16384
                                            // waves 1.17 ms, 4 and 8192 1.04, 8 and 4096 1.00, 16 and 2048 1.04)
constexpr uint32_t kLookupChunk = 32768;   // points per launch of a lookup in the box lists
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Pinned host memory for upload images.  Pinning new memory costs about 0.45 ms per MB, so blocks that
// are given back stay for the next image: at most kImageKeep of them and kImageKeepBytes, the
// smallest go first (the largest, where the bytes are too many).
constexpr size_t kImageKeep = 8, kImageKeepBytes = 16u << 20;
struct PinnedImage { char* mem = nullptr; size_t bytes = 0; };
std::mutex g_image_mu;
std::vector<PinnedImage> g_image_idle;      // by size

// most: the largest idle block to take for it.
int32_t take_image(size_t bytes, size_t most, PinnedImage& out) {
  {
    std::lock_guard<std::mutex> lock(g_image_mu);
    g_image_idle.reserve(kImageKeep + 1);   // (so that giving back allocates nothing)
    for (size_t i = 0; i < g_image_idle.size(); i++)
      if (g_image_idle[i].bytes >= bytes && g_image_idle[i].bytes <= most) {
        out = g_image_idle[i];
        g_image_idle.erase(g_image_idle.begin() + i);
        return MRL_OK;
      }
  }
  const size_t size = (bytes + 0xFFFF) & ~(size_t)0xFFFF;
  HIP_TRY(hipHostMalloc((void**)&out.mem, size, hipHostMallocPortable));
  out.bytes = size;
  return MRL_OK;
}

void give_image(PinnedImage& image) {
  if (!image.mem) return;
  PinnedImage drop[kImageKeep + 1];
  size_t n_drop = 0, total = image.bytes;
  {
    std::lock_guard<std::mutex> lock(g_image_mu);
    auto at = g_image_idle.begin();
    for (const PinnedImage& x : g_image_idle) { total += x.bytes; at += x.bytes < image.bytes; }
    g_image_idle.insert(at, image);
    while (total > kImageKeepBytes) { total -= g_image_idle.back().bytes; drop[n_drop++] = g_image_idle.back(); g_image_idle.pop_back(); }
    if (g_image_idle.size() > kImageKeep) { drop[n_drop++] = g_image_idle.front(); g_image_idle.erase(g_image_idle.begin()); }
  }
  for (size_t i = 0; i < n_drop; i++) (void)hipHostFree(drop[i].mem);
  image = PinnedImage();
}

struct ImageLease {
  PinnedImage image;
  ~ImageLease() { give_image(image); }
};

// Host-side compiled lattice: everything derived from (target, lattice).
struct Compiled {
  DevParams P;
  std::vector<TileEntry> tiles;
  std::vector<uint32_t> level_shapes;     // shapes grouped by dependency level, ascending inside a level
  std::vector<uint32_t> level_off;        // [n_levels + 1]
  std::vector<uint32_t> sizes[4];
  Geo geo;
  uint32_t merge_order[16];
  uint32_t n_shapes;
  uint64_t n_specs;
  std::vector<uint8_t> mk_entry;          // [256][V]
  std::vector<uint32_t> qdec;             // [Q] the axes of every bound vector, a byte each
  int lay_axis[5], dt_axis[5];            // coordinate axis of the operand's bit, -1 if none
  mrl_target_desc target;
  mrl_lattice_desc lat;                   // sizes pointers re-pointed to this->sizes
  // Pinned image of what a solve uploads (counters .. qdec), patched per call (device pointers).  The
  // first solve borrows a block for it, the second one keeps its own: many targets are solved once.
  mutable PinnedImage staging;
  mutable bool solved = false;
  mutable std::mutex solve_mu;            // solves of one compiled lattice take turns (they share the image)
  ~Compiled() { give_image(staging); }
};

// Offsets of the fixed part of the scratch buffer.
struct FixedLayout {
  size_t counters, params, tiles, level_shapes, level_off, mk_entry, blk_off, qdec, recs, masks, unit_cnt, unit_seg, bind, list, fitmap, maskD, maskC, mask2D, mask2C, colD, colC, lineD, lineC, prefD, prefC, tile_tmp, tile_tmp2, totals,
      upload_end, fill_end, end;
  uint32_t n_words;
  // the merge word by word (row_geo): its fixed lists from `shared` on, then dyn
  size_t shared, rows_rows, rows_first, rows_info, rows_cnt, rows_start, rows_sum, rows_tot, rows_dyn;
  // a solve's least: the fill's buffers share their place with the compression's and its lists
  size_t least() const { return fill_end > end ? fill_end : end; }
  size_t image_bytes() const { return upload_end - counters; }          // of what is uploaded, in pinned memory
};

// Whether the pass on the second merge axis a1 runs on the cells, before the boxes are made: the
// first axis a0 and a1 have strides of whole mask words, a1 lies outside a0 and has at most 64 steps.
bool second_on_cells(const Compiled& c, uint32_t* a0_out, uint32_t* a1_out) {
  const Geo& g = c.geo;
  uint32_t a0 = 0, a1 = 0, found = 0;
  for (uint32_t q = 0; q < g.ndim && found < 2; q++) {
    const uint32_t a = c.merge_order[q];
    if (g.ext[a] <= 1) continue;
    if (found++ == 0) a0 = a; else a1 = a;
  }
  if (a0_out) *a0_out = a0;
  if (a1_out) *a1_out = a1;
  return kSecondOnCells && found == 2 && g.stride[a0] % 64 == 0 && g.stride[a1] % (g.stride[a0] * g.ext[a0]) == 0 && g.ext[a1] <= 64;
}

// Entries of the table of alloc-binding costs (bind_kernel): read-only and accumulated operands of
// every size pair of the Move table.
size_t bind_entries(const Compiled& c) {
  return 2 * c.sizes[1].size() * c.sizes[3].size() * c.P.bind_d * ((size_t)6 << (2 * c.P.yb));
}

// Whether the table's boxes are merged word by word (rowmerge.hip) and its geometry there: the fit map comes from the
// plan, the size axes are merged first, there are four memory levels, a shape is one to kRowShapeWords mask words, and a
// row has at most 64 steps.  Rows lie along n, or along the first of k, m and b that has more than one step if those before it
// have not: a wave per row of one step is mostly waiting (b, m and k of 64, 64 and 16 sizes and one along n: 743 to 774 us
// box by box, 899 by words in rows of one, 675 in rows of 16).  Tables of four levels with 1 to 64 steps along n, everything or
// little fitting, 64 to 450 M cells, up to 255 sizes along k, m and b: the whole solve is 1.0 to 1.9 times as fast by words.
// may_turn: false for rows along n all the same, which the scratch may hold where it does not hold the turned ones: these are
// kept whole along k and dropped along m, and so can be more words (2 sizes along m, 57 along k, little fits: 3.5 instead of 2.1 MB).
bool row_geo(const Compiled& c, bool may_turn, RowGeo& g) {
  const DevParams& P = c.P;
  memset(&g, 0, sizeof g);
  if (P.gather || P.NL != 4 || P.log2V > 6 || c.n_specs >= (1ull << 31) || P.G % 64 || P.G / 64 > kRowShapeWords || P.nsz[3] > 64) return false;
  uint32_t turn = 0;
  while (may_turn && turn < 3 && P.nsz[3 - turn] == 1 && P.nsz[2 - turn] <= 64) turn++;
  for (uint32_t d = 0; d < 4; d++) g.axis[d] = (d + 4 - turn) & 3;
  g.en = P.nsz[g.axis[3]]; g.ek = P.nsz[g.axis[2]]; g.em = P.nsz[g.axis[1]]; g.eb = P.nsz[g.axis[0]];
  g.G = P.G; g.nw = P.G / 64;
  while ((1u << g.lg_nw) < g.nw) g.lg_nw++;
  g.n_shapes = c.n_shapes;
  g.n_planes = g.eb * g.em * g.nw;
  g.lv = P.log2V; g.ndt = P.ndt;
  g.n_levels = g.n_inner = P.nlv; g.level_axis = 3 + P.nlv;
  for (uint32_t a = 4 + P.nlv; a < c.geo.ndim; a++) {
    uint32_t bit = 0;
    while ((1u << bit) < c.geo.stride[a]) bit++;
    g.var_first |= 1u << bit;
    g.n_inner++;
    if (c.geo.ext[a] == 4) g.var_two |= 1u << bit;
    g.var_axis[bit] = a;
  }
  return true;
}

FixedLayout fixed_layout(const Compiled& c, bool may_turn = true) {
  FixedLayout f;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
  f.n_words = (uint32_t)((c.n_specs + 63) / 64);
  f.fitmap = take((size_t)f.n_words * 8 + 16);
  // uploaded in one copy: counters (zero), parameters, tile lists, level lists, microkernel table, bound vectors
  f.counters = take(sizeof(Counters));
  f.params = take(sizeof(DevParams));
  // From here on up to fill_end lies what the fill alone needs, and over it the compression's masks
  // and lists, which are written when the fill has ended: an 80-byte record per shape would otherwise
  // be 6 % of what a solve of a lattice with two memory levels asks for.
  const size_t shared = f.shared = o;
  f.tiles = take(c.tiles.size() * (c.P.gather ? sizeof(TileEntry) : sizeof(TileStep)) + 8);
  f.level_shapes = take(c.level_shapes.size() * 4);
  f.level_off = take(c.level_off.size() * 4);
  f.blk_off = c.P.gather ? 0 : take(c.level_off.size() * 4);
  f.mk_entry = take(c.mk_entry.size());
  f.qdec = take(c.qdec.size() * 4);
  f.upload_end = o;
  const size_t n_items = (size_t)c.n_shapes * c.P.npass;
  f.recs = f.masks = f.unit_cnt = f.unit_seg = f.bind = f.list = 0;
  if (!c.P.gather) {
    const uint32_t n_lev = (uint32_t)c.level_off.size() - 1;
    f.masks = take(n_items * ((size_t)c.P.nwp << c.P.ndt) * 8);
    f.recs = take(plan_bytes_recs(c.n_shapes));
    f.unit_cnt = take((size_t)unit_blocks(c.level_off.data(), n_lev, c.P.npass, nullptr) * c.P.nranks * 4);
    f.unit_seg = take(((size_t)n_lev * c.P.nranks + 1) * 4);
    if (c.P.moves) f.bind = take(bind_entries(c) * 8);
    // the work list takes what is left of the buffer; where that is less than the whole list, it goes through in windows
    f.list = take(std::max<size_t>(n_items, 64) * 8);
  }
  f.fill_end = o;
  o = shared;
  f.maskD = take((size_t)f.n_words * 8);
  f.maskC = take((size_t)f.n_words * 8);
  f.mask2D = f.mask2C = f.colD = f.colC = 0;
  if (second_on_cells(c, nullptr, nullptr)) {
    uint32_t a1 = 0;
    second_on_cells(c, nullptr, &a1);
    f.mask2D = take((size_t)f.n_words * 8);
    f.mask2C = take((size_t)f.n_words * 8);
    f.colD = take((size_t)(c.n_specs / c.geo.ext[a1]) * 8);
    f.colC = take((size_t)(c.n_specs / c.geo.ext[a1]) * 8);
  }
  {
    // line-major copies of the two masks: one bit per cell, 64-bit words per line of the first merge axis
    uint32_t e0 = c.geo.ext[c.merge_order[0]];
    for (uint32_t q = 0; q < c.geo.ndim; q++) if (c.geo.ext[c.merge_order[q]] > 1) { e0 = c.geo.ext[c.merge_order[q]]; break; }
    const size_t line_bytes = (size_t)(c.n_specs / e0) * ((e0 + 63) / 64) * 8;
    f.lineD = take(line_bytes);
    f.lineC = take(line_bytes);
  }
  f.prefD = take((size_t)f.n_words * 4);
  f.prefC = take((size_t)f.n_words * 4);
  f.tile_tmp = take((c.n_specs / kScanTileItems + 2) * 4);
  f.tile_tmp2 = take((c.n_specs / kScanTileItems + 2) * 4);
  f.totals = take(64);
  f.end = o;
  RowGeo g;
  f.rows_rows = f.rows_first = f.rows_info = f.rows_cnt = f.rows_start = f.rows_sum = f.rows_tot = f.rows_dyn = 0;
  if (row_geo(c, may_turn, g)) {
    o = shared;
    f.rows_rows = take((size_t)g.n_planes * 4);
    f.rows_first = take((size_t)g.n_planes * 4);
    f.rows_info = take((size_t)g.n_planes * g.ek * kRowInfoBytes);
    f.rows_cnt = take((size_t)g.n_shapes * 8);
    f.rows_start = take((size_t)g.n_shapes * 8);
    f.rows_sum = take(rows_sum_bytes(g));
    f.rows_tot = take(kRowTotals * 4);
    f.rows_dyn = o;
  }
  return f;
}

// per box while merging: bcell, blen, alive, next, pos, and for the dense copies of the live boxes
// cell2, len2, alive2, pos2; a flag per 256 boxes.  Per final box: fcell, flen, fv0, fv1
size_t work_bytes(uint64_t nb) { return 5 * align_up(nb * 4) + 2 * align_up(nb * 16) + 2 * align_up(nb) + align_up((nb / 256 + 1) * 4); }
size_t final_bytes(uint64_t nb) { return align_up(nb * 4) + align_up(nb * 16) + 2 * align_up(nb * 8); }

uint32_t ipow(uint32_t b, uint32_t e) { uint32_t r = 1; while (e--) r *= b; return r; }

int32_t validate_target(const mrl_target_desc* d) {
  if (!d) return fail(MRL_E_INVAL, "target descriptor is NULL");
  if (d->n_levels < 1 || d->n_levels > MRL_MAX_LEVELS) return fail(MRL_E_INVAL, "n_levels must be 1..4");
  if (d->n_microkernels > MRL_MAX_MK) return fail(MRL_E_INVAL, "too many microkernels");
  for (uint32_t j = 0; j < d->n_microkernels; j++) {
    if (d->mk[j].kind > MRL_MK_VEC_RELU) return fail(MRL_E_INVAL, "unknown microkernel kind %u", d->mk[j].kind);
    if (d->mk[j].lanes < 1) return fail(MRL_E_INVAL, "microkernel lanes must be >= 1");
    if (d->mk[j].kind != MRL_MK_SCALAR_FMA && d->mk[j].kind != MRL_MK_SCALAR_ADDRELU && d->mk[j].kind != MRL_MK_SCALAR_MOVE &&
        d->mk[j].kind != MRL_MK_SCALAR_ADD && d->mk[j].kind != MRL_MK_SCALAR_RELU && d->n_levels < 2)
      return fail(MRL_E_INVAL, "vector microkernels need a level 1");
  }
  return MRL_OK;
}

int32_t compile(const mrl_target_desc& T, const mrl_lattice_desc* L, Compiled& c) {
  if (!L) return fail(MRL_E_INVAL, "lattice descriptor is NULL");
  if (L->kind > MRL_KIND_BIAS_ADD_RELU_SPLIT) return fail(MRL_E_INVAL, "unknown spec kind %u", L->kind);
  // A parallel lattice is a Matmul lattice (same operator, operands and coordinates) with more
  // rewrites; a bounded one is the lattice of its operator with more coordinates; a Matmul whose
  // Moves are Move Specs is a Matmul lattice with other Move costs; the composition of two Matmuls
  // has the fused Spec's structure (four operands and an intermediate between two stages).
  const bool chain = L->kind == MRL_KIND_MATMUL_CHAIN;
  // The bias add alone has the operands and coordinates of the bias-add + ReLU (other microkernels
  // apply to it); the ReLU alone has two tensors; the bias-add + ReLU with its own bufferize has
  // more rewrites.
  const bool add_only = L->kind == MRL_KIND_BIAS_ADD, relu_only = L->kind == MRL_KIND_RELU, split = L->kind == MRL_KIND_BIAS_ADD_RELU_SPLIT;
  const bool parallel = L->kind == MRL_KIND_MATMUL_PARALLEL, move_specs = L->kind == MRL_KIND_MOVE, moves = L->kind == MRL_KIND_MATMUL_MOVES;
  const bool bounded = L->kind >= MRL_KIND_MATMUL_BOUNDED && L->kind <= MRL_KIND_FUSED_BOUNDED;
  const uint32_t kind = parallel || moves ? (uint32_t)kKindM : bounded ? L->kind - MRL_KIND_MATMUL_BOUNDED : move_specs ? (uint32_t)kKindV
                        : chain ? (uint32_t)kKindF : add_only || split ? (uint32_t)kKindE : relu_only ? (uint32_t)kKindR : L->kind;
  if (parallel && T.threads < 1) return fail(MRL_E_INVAL, "a MATMUL_PARALLEL lattice needs threads >= 1");
  if ((move_specs || moves) && T.line_bytes < 1) return fail(MRL_E_INVAL, "MOVE and MATMUL_MOVES lattices need line_bytes >= 1");
  c.target = T;
  c.lat = *L;
  DevParams& P = c.P;
  memset(&P, 0, sizeof P);
  P.kind = kind;
  P.par = parallel ? 1u : 0u;
  P.threads = parallel ? T.threads : 1u;
  P.sync = T.sync_cost;
  // memory bounds: one axis per level of finite capacity, values 0, 1, 2, 4, ... up to the capacity
  P.bounded = bounded ? 1u : 0u;
  P.Q = 1;
  for (uint32_t l = 0; l < 4; l++) P.lim_of_level[l] = kNoBit;
  if (bounded) {
    for (uint32_t l = 0; l < T.n_levels; l++) {
      if (T.capacity_bytes[l] == UINT64_MAX) continue;
      uint32_t nq = 1;
      while (nq < 64 && (1ull << (nq - 1)) <= T.capacity_bytes[l]) nq++;
      P.lim_of_level[l] = P.nlim;
      P.lim_nq[P.nlim++] = nq;
    }
  }
  bool packed = false;       // some tensor may be packed in strips
  for (uint32_t i = 0; i < 5; i++) {
    if (L->layout_coord[i] > 2) return fail(MRL_E_INVAL, "layout_coord[%u] must be 0, 1 or 2", i);
    if (L->layout_coord[i] == 2) {
      if (!(move_specs || moves)) return fail(MRL_E_INVAL, "packed layouts (layout_coord 2) only in MOVE and MATMUL_MOVES lattices");
      if (T.strip < 2 || T.strip % 2) return fail(MRL_E_INVAL, "packed layouts need an even strip >= 2");
      packed = true;
    }
  }
  P.strip = T.strip;
  P.xw = packed ? 4u : 2u;
  if (move_specs) {
    // contiguousness (a packed tensor has three physical dimensions) and aligned flag of the source, then of the destination
    P.nlim = 4;
    P.lim_nq[0] = packed ? 4 : 3; P.lim_nq[1] = 2; P.lim_nq[2] = packed ? 4 : 3; P.lim_nq[3] = 2;
  }
  for (uint32_t a = P.nlim; a-- > 0;) { P.lim_stride[a] = P.Q; P.Q *= P.lim_nq[a]; }
  P.gather = bounded || move_specs ? 1u : 0u;
  P.bind_d = 1;
  for (uint32_t i = 0; i < 3; i++) if (L->dtype_coord[i] || L->base_dtype_bytes[i] == 2) P.bind_d = 3;
  P.yb = packed ? 2 : 1;
  P.moves = moves ? 1u : 0u;
  P.chain = chain ? 1u : 0u;
  P.split = split ? 1u : 0u;
  P.line_bytes = T.line_bytes;
  P.line_mask = T.line_bytes && (T.line_bytes & (T.line_bytes - 1)) == 0 ? T.line_bytes - 1 : 0;
  for (int l = 0; l < 4; l++) P.weight[l] = T.level_weight[l];
  P.nops = kind == kKindF ? 4 : kind == kKindV || kind == kKindR ? 2 : 3;
  P.nlv = kind == kKindF ? 5 : kind == kKindV || kind == kKindR ? 2 : 3;
  P.NL = T.n_levels;
  P.npass = kind == kKindF ? P.NL : 1;
  P.ncombo = ipow(P.NL, P.nops);
  uint64_t max_vol = 1;
  uint32_t maxs = 0;
  for (int d = 0; d < 4; d++) {
    uint32_t n = L->n_sizes[d];
    if (n < 1 || n > MRL_MAX_SIZES || !L->sizes[d]) return fail(MRL_E_INVAL, "n_sizes[%d] must be 1..%d", d, MRL_MAX_SIZES);
    c.sizes[d].assign(L->sizes[d], L->sizes[d] + n);
    // (no rewrite of a fused Spec changes k: a fused lattice may cover any stretch of k values)
    if (c.sizes[d][0] != 1 && !(d == 2 && kind == kKindF && !chain)) return fail(MRL_E_INVAL, "sizes[%d] must start with 1", d);
    for (uint32_t j = 1; j < n; j++)
      if (c.sizes[d][j] <= c.sizes[d][j - 1]) return fail(MRL_E_INVAL, "sizes[%d] must be strictly ascending", d);
    c.lat.sizes[d] = c.sizes[d].data();
    P.nsz[d] = n;
    for (uint32_t j = 0; j < n; j++) P.sizes[d][j] = c.sizes[d][j];
    max_vol *= c.sizes[d][n - 1];
    if (max_vol >= (1ull << 48)) return fail(MRL_E_INVAL, "b*m*k*n must stay below 2^48");
    maxs = std::max(maxs, n);
  }
  if (kind != kKindM && !chain && L->n_sizes[0] != 1) return fail(MRL_E_INVAL, "this kind has no batch dimension");
  if ((kind == kKindE || kind == kKindR) && L->n_sizes[2] != 1) return fail(MRL_E_INVAL, "BIAS_ADD_RELU, BIAS_ADD and RELU have no k dimension");
  if (kind == kKindV && L->n_sizes[2] != 1) return fail(MRL_E_INVAL, "MOVE has no k dimension");
  if (moves && L->n_sizes[0] != 1) return fail(MRL_E_INVAL, "MATMUL_MOVES has no batch dimension");
  P.shape_stride[3] = 1;
  for (int d = 2; d >= 0; d--) P.shape_stride[d] = P.shape_stride[d + 1] * P.nsz[d + 1];
  c.n_shapes = P.shape_stride[0] * P.nsz[0];

  // variant bits: layout bits (operand order) above dtype bits (operand order)
  for (int i = 0; i < 5; i++) { P.lay_bit[i] = P.dt_bit[i] = kNoBit; c.lay_axis[i] = c.dt_axis[i] = -1; }
  for (uint32_t i = 0; i < P.nops; i++) {
    P.nlay += L->layout_coord[i];          // bits of the layout field
    P.lay_w[i] = L->layout_coord[i];
    P.ndt += L->dtype_coord[i] ? 1 : 0;
    if (L->dtype_coord[i] && !(kind == kKindV || (kind == kKindM && i < 2))) return fail(MRL_E_INVAL, "dtype bit only on MatmulAccum inputs and on the tensors of a MOVE");
    if (L->base_dtype_bytes[i] != 4 && !(L->base_dtype_bytes[i] == 2 && (kind == kKindM || kind == kKindV)))
      return fail(MRL_E_INVAL, "base_dtype_bytes[%u] must be 4 (or 2 on a MatmulAccum or a MOVE)", i);
    P.base_bf16[i] = L->base_dtype_bytes[i] == 2;
    // (the second Matmul of a composition accumulates into out, as every Matmul does)
    P.access[i] = kind == kKindM ? (i == 2 ? kRmw : kRead) : (i == P.nops - 1 ? (chain ? kRmw : kWrite) : kRead);
    P.lvpow[i] = ipow(P.NL, P.nops - 1 - i);
    P.pack_shift[i] = 2 * (P.nops - 1 - i);
  }
  P.V = 1u << (P.nlay + P.ndt);
  P.log2V = P.nlay + P.ndt;

  if (P.V > (P.gather || P.moves ? 64u : 16u)) return fail(MRL_E_INVAL, "too many layout/dtype bits");
  {
    uint32_t axis = 4 + P.nlv + P.nlim, seen_l = 0, seen_d = 0;
    for (uint32_t i = 0; i < P.nops; i++)
      if (L->layout_coord[i]) { seen_l += L->layout_coord[i]; c.lay_axis[i] = (int)axis++; P.lay_bit[i] = P.ndt + P.nlay - seen_l; }
    for (uint32_t i = 0; i < P.nops; i++)
      if (L->dtype_coord[i]) { c.dt_axis[i] = (int)axis++; P.dt_bit[i] = P.ndt - 1 - seen_d++; }
  }
  if ((uint64_t)P.ncombo * P.npass * P.V * P.Q >= (1ull << 32)) return fail(MRL_E_INVAL, "too many entries per shape");
  P.G = P.ncombo * P.npass * P.V * P.Q;
  c.n_specs = (uint64_t)c.n_shapes * P.G;
  if (c.n_specs < (1ull << 32) && P.nlim) {
    c.qdec.resize(P.Q);
    for (uint32_t q = 0; q < P.Q; q++) {
      c.qdec[q] = 0;
      for (uint32_t a = 0; a < P.nlim; a++) c.qdec[q] |= (q / P.lim_stride[a] % P.lim_nq[a]) << (8 * a);
    }
  }
  if (c.n_specs >= (1ull << 32)) return fail(MRL_E_INVAL, "lattice has %llu specs; the limit is 2^32-1", (unsigned long long)c.n_specs);

  for (uint32_t i = 0; i < P.nops; i++) {
    P.mstride[i] = (P.lvpow[i] * P.npass) << P.log2V;
    P.unit_lay += L->layout_coord[i] ? 1u : 0u;
  }

  // target
  for (int l = 0; l < 4; l++) {
    P.cap[l] = T.capacity_bytes[l];
    P.zero[l] = T.zero_coef[l];
  }
  P.convert = T.convert_coef;
  P.s = T.loop_overhead;
  P.nmk = T.n_microkernels;
  for (uint32_t j = 0; j < P.nmk; j++) { P.mk_kind[j] = T.mk[j].kind; P.mk_lanes[j] = T.mk[j].lanes; P.mk_cost[j] = T.mk[j].cost; }

  // rewrite ids
  P.maxs = maxs;
  P.move_base = P.nmk;
  P.tile_base = P.move_base + P.nops * (P.NL - 1) * 2 * P.xw;
  P.buf_id = P.tile_base + 4 * maxs;
  P.par_base = P.buf_id + 1;
  if ((parallel ? P.par_base + 4 * maxs : P.buf_id + P.NL) >= kNone) return fail(MRL_E_INVAL, "rewrite ids do not fit 16 bits");

  // Moves: coefficient per (operand, src, dst, transposed) and the list of Moves that can occur
  for (uint32_t i = 0; i < (move_specs || moves ? 0u : P.nops); i++)
    for (uint32_t src = 0; src < P.NL; src++)
      for (uint32_t dst = 0; dst < src; dst++)
        for (uint32_t x = 0; x < 2; x++) {
          if (x && !L->layout_coord[i]) continue;
          const uint32_t ld = T.load_coef[src][dst][x], st = T.store_coef[dst][src][x];
          uint64_t cf = 0;
          if (P.access[i] != kWrite) { if (!ld) continue; cf += ld; }
          if (P.access[i] != kRead) { if (!st) continue; cf += st; }
          if (cf > UINT32_MAX) return fail(MRL_E_INVAL, "Move coefficients too large");
          P.mcoef[i][src][dst][x] = (uint32_t)cf;
          P.mcoef[i][src][3][0] += cf ? 1u : 0u;
        }
  for (uint32_t i = 0; i < P.nops; i++) P.can_convert[i] = L->dtype_coord[i] && P.access[i] == kRead;
  {
    // (below 2^48 each: the volume is.  b holds p in a composition)
    const uint64_t b = c.sizes[0].back(), m = c.sizes[1].back(), k = c.sizes[2].back(), n = c.sizes[3].back(), mk = m * k, kn = k * n, mn = m * n;
    uint64_t most = std::max({mk, kn, mn}) * (chain ? 1 : b), coef = 0;
    if (chain) most = std::max({most, m * b, k * b, b * n});
    for (uint32_t i = 0; i < P.nops; i++)
      for (uint32_t src = 0; src < P.NL; src++)
        for (uint32_t dst = 0; dst < src; dst++)
          for (uint32_t x = 0; x < 2; x++) coef = std::max<uint64_t>(coef, P.mcoef[i][src][dst][x]);
    coef += P.convert;
    P.small = most <= UINT32_MAX && coef < (1u << 30) && c.n_specs < (1u << 29);
  }

  // microkernels: the level / layout / dtype part of each predicate, per (pack, variant)
  c.mk_entry.assign((size_t)256 * P.V, 0);
  for (uint32_t pack = 0; pack < 256; pack++)
    for (uint32_t v = 0; v < P.V; v++) {
      uint32_t lv[4], ly[4], bf[4];
      bool in_range = true;
      for (uint32_t i = 0; i < 4; i++) {
        lv[i] = i < P.nops ? (pack >> P.pack_shift[i]) & 3u : 0u;
        in_range = in_range && lv[i] < P.NL;
        ly[i] = i < P.nops && P.lay_bit[i] != kNoBit ? (v >> P.lay_bit[i]) & ((1u << P.lay_w[i]) - 1u) : 0u;
        bf[i] = i < P.nops ? (P.dt_bit[i] != kNoBit ? (v >> P.dt_bit[i]) & 1u : P.base_bf16[i]) : 0u;
      }
      if (!in_range || (P.nops < 4 && (pack >> (2 * P.nops)))) continue;
      uint8_t bits = 0;
      for (uint32_t j = 0; j < P.nmk; j++) {
        bool ok = false;
        const bool all_f32 = !(bf[0] | bf[1] | bf[2]);
        switch (T.mk[j].kind) {
          case MRL_MK_SCALAR_FMA: ok = P.kind == kKindM && !(lv[0] | lv[1] | lv[2]) && all_f32; break;
          case MRL_MK_BCAST_VEC_MULADD: {
            // rhs, out row-major; one row in whole packed strips is the same sequence of values
            auto rowlike = [&](uint32_t y) { return y == 0 || (y == 2 && T.strip % T.mk[j].lanes == 0); };
            ok = P.kind == kKindM && lv[0] == 0 && lv[1] == 1 && lv[2] == 1 && all_f32 && rowlike(ly[1]) && rowlike(ly[2]);
            break;
          }
          case MRL_MK_BF16_DOT: ok = P.kind == kKindM && lv[0] == 1 && lv[1] == 1 && lv[2] == 0 && bf[0] && bf[1] && !bf[2] && (P.lay_bit[1] == kNoBit || ly[1] == 1); break;
          case MRL_MK_SCALAR_ADDRELU: ok = P.kind == kKindE && !add_only && !(lv[0] | lv[1] | lv[2]); break;
          case MRL_MK_VEC_ADDRELU: ok = P.kind == kKindE && !add_only && lv[0] == 1 && lv[1] == 1 && lv[2] == 1 && !ly[0] && !ly[2]; break;
          case MRL_MK_SCALAR_ADD: ok = add_only && !(lv[0] | lv[1] | lv[2]); break;
          case MRL_MK_VEC_ADD: ok = add_only && lv[0] == 1 && lv[1] == 1 && lv[2] == 1 && !ly[0] && !ly[2]; break;
          case MRL_MK_SCALAR_RELU: ok = relu_only && !(lv[0] | lv[1]); break;
          case MRL_MK_VEC_RELU: ok = relu_only && lv[0] == 1 && lv[1] == 1 && !ly[0] && !ly[1]; break;
          // (the contiguousness / alignment part of the move microkernels' predicates is tested in the kernel)
          case MRL_MK_SCALAR_MOVE: ok = P.kind == kKindV && !(!bf[0] && bf[1]); break;
          case MRL_MK_VECTOR_MOVE:
          case MRL_MK_VECTOR_MOVE_ALIGNED:
            // (rows of strips: whether the strips are whole vectors is tested in the kernel, with the shape)
            ok = P.kind == kKindV && ((lv[0] == 1 && lv[1] > 1) || (lv[1] == 1 && lv[0] > 1)) && ly[0] != 1 && ly[1] != 1 &&
                 (ly[0] == 3) == (ly[1] == 3) && bf[0] == bf[1];
            break;
        }
        bits |= (uint8_t)((ok ? 1u : 0u) << j);
      }
      c.mk_entry[(size_t)pack * P.V + v] = bits;
    }

  // tiles: for (dim, size index) the smaller allowed sizes dividing it
  for (int d = 0; d < 4; d++) {
    P.tile_dim_ok[d] = kind == kKindM || d == 1 || d == 3;
    for (uint32_t j = 0; j < P.nsz[d]; j++) {
      P.tile_off[d][j] = (uint32_t)c.tiles.size();
      if (P.tile_dim_ok[d])
        for (uint32_t jt = 0; jt < j; jt++)
          if (c.sizes[d][j] % c.sizes[d][jt] == 0) {
            c.tiles.push_back(TileEntry{jt, c.sizes[d][j] / c.sizes[d][jt]});
          }
    }
    for (uint32_t j = P.nsz[d]; j <= (uint32_t)kMaxSizes; j++) P.tile_off[d][j] = (uint32_t)c.tiles.size();
  }

  // operand-level combos by rank
  P.nwp = (P.ncombo + 63) / 64;
  P.nranks = P.nops * (P.NL - 1) + 1;
  {
    std::vector<std::pair<uint32_t, uint32_t>> order;
    for (uint32_t combo = 0; combo < P.ncombo; combo++) {
      uint32_t r = 0, x = combo;
      for (uint32_t i = 0; i < P.nops; i++) { r += x % P.NL; x /= P.NL; }
      order.push_back({r, combo});
    }
    std::sort(order.begin(), order.end());
    uint32_t q = 0;
    for (uint32_t r = 0; r <= P.nranks; r++) {
      while (q < order.size() && order[q].first < r) q++;
      P.rank_off[r] = q;
    }
    for (uint32_t i = 0; i < order.size(); i++) {
      const uint32_t combo = order[i].second;
      uint32_t pack = 0;
      for (uint32_t op = 0; op < P.nops; op++) pack |= ((combo / P.lvpow[op]) % P.NL) << P.pack_shift[op];
      uint32_t info = pack;
      for (uint32_t op = 0; op < P.nops; op++) info |= 1u << (8 + 4 * ((combo / P.lvpow[op]) % P.NL) + op);
      P.combo_info[P.gather ? i : combo] = info;
      P.rank_mask[order[i].first][combo >> 6] |= 1ull << (combo & 63);
    }
  }

  // dependency level of a shape = sum over tiled dims of the longest divisor chain below its size
  std::vector<uint32_t> depth[4];
  uint32_t n_lev = 1;
  for (int d = 0; d < 4; d++) {
    depth[d].assign(P.nsz[d], 0);
    uint32_t mx = 0;
    if (P.tile_dim_ok[d])
      for (uint32_t j = 0; j < P.nsz[d]; j++) {
        for (uint32_t q = P.tile_off[d][j]; q < P.tile_off[d][j + 1]; q++)
          depth[d][j] = std::max(depth[d][j], depth[d][c.tiles[q].jt] + 1);
        mx = std::max(mx, depth[d][j]);
      }
    n_lev += mx;
  }
  std::vector<uint32_t> lev(c.n_shapes);
  c.level_off.assign(n_lev + 1, 0);
  for (uint32_t sh = 0; sh < c.n_shapes; sh++) {
    uint32_t r = sh, l = 0;
    for (int d = 0; d < 4; d++) { l += depth[d][r / P.shape_stride[d]]; r %= P.shape_stride[d]; }
    lev[sh] = l;
    c.level_off[l + 1]++;
  }
  for (uint32_t l = 0; l < n_lev; l++) c.level_off[l + 1] += c.level_off[l];
  c.level_shapes.resize(c.n_shapes);
  {
    std::vector<uint32_t> cur(c.level_off.begin(), c.level_off.end() - 1);
    for (uint32_t sh = 0; sh < c.n_shapes; sh++) c.level_shapes[cur[lev[sh]]++] = sh;
  }

  // coordinate geometry and merge order: the memory-bound axes, n, k, m, b, the level axes,
  // layout bits, dtype bits, each group from its last axis to its first
  Geo& g = c.geo;
  memset(&g, 0, sizeof g);
  uint32_t nd = 0;
  for (int d = 0; d < 4; d++) g.ext[nd++] = P.nsz[d];
  for (uint32_t i = 0; i < P.nlv; i++) g.ext[nd++] = P.NL;
  for (uint32_t a = 0; a < P.nlim; a++) g.ext[nd++] = P.lim_nq[a];
  for (uint32_t i = 0; i < P.nops; i++) if (L->layout_coord[i]) g.ext[nd++] = 1u << L->layout_coord[i];
  for (uint32_t i = 0; i < P.ndt; i++) g.ext[nd++] = 2;
  if (nd > 16) return fail(MRL_E_INVAL, "more than 16 coordinate axes");
  g.ndim = nd;
  uint64_t s = 1;
  for (int a = (int)nd - 1; a >= 0; a--) { g.stride[a] = (uint32_t)s; s *= g.ext[a]; }
  g.n = (uint32_t)c.n_specs;
  {
    uint32_t q = 0;
    const int lim0 = 4 + (int)P.nlv, lay0 = lim0 + (int)P.nlim;
    for (int a = lay0 - 1; a >= lim0; a--) c.merge_order[q++] = (uint32_t)a;             // memory bounds
    for (int a = 3; a >= 0; a--) c.merge_order[q++] = (uint32_t)a;                       // n, k, m, b
    for (int a = lim0 - 1; a >= 4; a--) c.merge_order[q++] = (uint32_t)a;                // levels
    int n_lay_axes = 0;
    for (uint32_t i = 0; i < P.nops; i++) n_lay_axes += L->layout_coord[i] ? 1 : 0;
    for (int a = lay0 + n_lay_axes - 1; a >= lay0; a--) c.merge_order[q++] = (uint32_t)a;
    for (int a = (int)nd - 1; a >= lay0 + n_lay_axes; a--) c.merge_order[q++] = (uint32_t)a;
  }

  return MRL_OK;
}


// compile() costs up to a few milliseconds for the larger lattices; repeated solves of the same
// (target, lattice) reuse the result.  Entries are immutable once published; the least recently used
// goes first.  A program that takes turns between a few targets keeps all of its lattices: up to
// kCompiledMost of them within kCompiledBytes, and kCompiledLeast however large they are (config 5 has
// three lattices; with 8 entries, first in first out, three targets in turn compiled all of them in every
// step: 6.8 instead of 5.4 ms.  That helps a program which comes back to a target; a target's first
// solve compiles its lattices as ever).
constexpr size_t kCompiledMost = 32, kCompiledLeast = 8;
constexpr size_t kCompiledBytes = 64u << 20;
using CompiledPtr = std::shared_ptr<const Compiled>;

bool same_problem(const Compiled& c, const mrl_target_desc& T, const mrl_lattice_desc& L) {
  // (the whole target is compared, also the fields this lattice's kind does not use)
  if (memcmp(&c.target, &T, sizeof T) || c.lat.kind != L.kind) return false;
  if (memcmp(c.lat.layout_coord, L.layout_coord, sizeof L.layout_coord) ||
      memcmp(c.lat.dtype_coord, L.dtype_coord, sizeof L.dtype_coord) ||
      memcmp(c.lat.base_dtype_bytes, L.base_dtype_bytes, sizeof L.base_dtype_bytes)) return false;
  for (int d = 0; d < 4; d++) {
    if (L.n_sizes[d] != c.sizes[d].size() || !L.sizes[d]) return false;
    if (memcmp(L.sizes[d], c.sizes[d].data(), c.sizes[d].size() * sizeof(uint32_t))) return false;
  }
  return true;
}

int32_t get_compiled(const mrl_target_desc& T, const mrl_lattice_desc* L, CompiledPtr& out) {
  static std::mutex mu;
  static std::vector<CompiledPtr> cache;          // most recently used last
  if (L && L->kind <= MRL_KIND_BIAS_ADD_RELU_SPLIT) {
    std::lock_guard<std::mutex> lock(mu);
    for (size_t i = cache.size(); i-- > 0;)
      if (same_problem(*cache[i], T, *L)) {
        std::rotate(cache.begin() + i, cache.begin() + i + 1, cache.end());
        out = cache.back();
        return MRL_OK;
      }
  }
  auto c = std::make_shared<Compiled>();
  const int32_t rc = compile(T, L, *c);
  if (rc) return rc;
  std::lock_guard<std::mutex> lock(mu);
  cache.push_back(c);
  out = c;
  // what an entry holds: its lists, and from its first solve on their image in pinned memory
  size_t bytes = 0;
  for (const CompiledPtr& e : cache) bytes += 2 * fixed_layout(*e).image_bytes();
  while (cache.size() > kCompiledMost || (cache.size() > kCompiledLeast && bytes > kCompiledBytes)) {
    bytes -= 2 * fixed_layout(*cache.front()).image_bytes();
    cache.erase(cache.begin());
  }
  return MRL_OK;
}

// A second stream (default priority, non-blocking) for work that is independent of what runs on
// the caller's stream: one of the two box lists beside the other; with it the events and the pinned counters a solve needs.
// u32: 16 for the box lists, then the diagonals' first places in the work list (at most 62), then the counters (a copy to memory
// that is not pinned goes through a staging buffer and waits for it)
constexpr size_t kDiagFirst = 16, kCountersAt = kDiagFirst + 64, kPinnedCounts = kCountersAt + sizeof(Counters) / 4;
struct Aux {
  hipStream_t stream = nullptr;
  std::vector<hipEvent_t> events;
  uint32_t* h_counts = nullptr;     // pinned: counts read back without stalling the other stream
  hipEvent_t timing[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};   // fill start, fill end, compression end and start, plan + pre-fill end, first dependency level
  int device = -1;
  bool busy = false;
};

// One set per solve in flight (solves on different host threads may overlap; a box list that is taken
// to the host uses the stream of one), kept for reuse.
struct AuxLease {
  Aux* a = nullptr;
  ~AuxLease();
};
std::mutex g_aux_mu;
std::vector<std::unique_ptr<Aux>> g_aux_pool;
AuxLease::~AuxLease() {
  if (a) { std::lock_guard<std::mutex> lock(g_aux_mu); a->busy = false; }
}

int32_t get_aux(size_t n_events, AuxLease& lease) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  Aux* aux = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_aux_mu);
    for (auto& p : g_aux_pool) if (!p->busy && p->device == dev) { aux = p.get(); break; }
    if (!aux) {
      g_aux_pool.emplace_back(new Aux);
      aux = g_aux_pool.back().get();
      aux->device = dev;
    }
    aux->busy = true;
  }
  lease.a = aux;
  if (!aux->stream) HIP_TRY(hipStreamCreateWithFlags(&aux->stream, hipStreamNonBlocking));
  if (!aux->h_counts) HIP_TRY(hipHostMalloc((void**)&aux->h_counts, kPinnedCounts * 4, hipHostMallocDefault));
  for (auto& e : aux->timing) if (!e) HIP_TRY(hipEventCreate(&e));
  while (aux->events.size() < n_events) {
    hipEvent_t e;
    HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    aux->events.push_back(e);
  }
  return MRL_OK;
}

// Pinned host memory through which a call exchanges data with the GPU, in two halves: the kernels
// read and write it in place (no copy commands), one half while the host works on the other.
// Blocks are kept for the next call, at most kStageKeep of them idle.
constexpr size_t kStageHalf = 2u << 20;
constexpr size_t kStageKeep = 4;
std::mutex g_stage_mu;
std::vector<char*> g_stage_idle;

struct StageLease {
  char* mem = nullptr;
  ~StageLease() {
    if (!mem) return;
    {
      std::lock_guard<std::mutex> lock(g_stage_mu);
      if (g_stage_idle.size() < kStageKeep) {          // (room for kStageKeep is reserved below)
        g_stage_idle.push_back(mem);
        return;
      }
    }
    (void)hipHostFree(mem);
  }
};

int32_t get_stage(StageLease& lease) {
  {
    std::lock_guard<std::mutex> lock(g_stage_mu);
    g_stage_idle.reserve(kStageKeep);
    if (!g_stage_idle.empty()) {
      lease.mem = g_stage_idle.back();
      g_stage_idle.pop_back();
      return MRL_OK;
    }
  }
  HIP_TRY(hipHostMalloc((void**)&lease.mem, 2 * kStageHalf, hipHostMallocPortable | hipHostMallocMapped));
  return MRL_OK;
}

// Makes a device current for a scope: a question may be asked while another one is.  The null stream is the current
// device's, and so are a helper stream and an event, which is recorded on streams of its own device only.
struct OnDevice {
  int before = -1;
  int32_t set(int device) {
    int now = 0;
    HIP_TRY(hipGetDevice(&now));
    if (now == device) return MRL_OK;
    HIP_TRY(hipSetDevice(device));
    before = now;
    return MRL_OK;
  }
  ~OnDevice() { if (before >= 0) (void)hipSetDevice(before); }
};

// Host threads that run the jobs of mrl_solve_graph and stretches of long questions.  They are kept
// between calls (a thread's first HIP calls are slow) and never end; every queued task gets a thread,
// since tasks wait for each other.  The pool is never destroyed: its threads may still wait in it
// when the process ends.
class Workers {
 public:
  void submit(std::function<void()> task) {
    std::lock_guard<std::mutex> lk(mu_);
    queue_.push_back(std::move(task));
    if (idle_ < queue_.size()) {
      try { std::thread([this] { loop(); }).detach(); }
      catch (...) { queue_.pop_back(); throw; }
    }
    cv_.notify_all();
  }

 private:
  void loop() {
    for (;;) {
      std::function<void()> task;
      {
        std::unique_lock<std::mutex> lk(mu_);
        idle_++;
        cv_.wait(lk, [&] { return !queue_.empty(); });
        idle_--;
        task = std::move(queue_.front());
        queue_.erase(queue_.begin());
      }
      task();
    }
  }
  std::mutex mu_;
  std::condition_variable cv_;
  std::vector<std::function<void()>> queue_;
  size_t idle_ = 0;
};
Workers& workers() { static Workers* w = new Workers; return *w; }

// Take n items through the GPU, `chunk` at a time, on `stream`: fill(first, m, half) writes a chunk's
// inputs, launch(first, m, half) queues its kernel and drain(first, m, half) takes its results.  While
// the GPU has one chunk the host drains the one before it and fills the next.  When this returns,
// with or without an error, nothing queued here is still running.
struct StageHalves {
  char* mem;
  size_t bytes;
  char* half(size_t i) const { return mem + (i & 1) * bytes; }
};
template <class Fill, class Launch, class Drain>
int32_t take_through(size_t n, size_t chunk, const StageHalves& stage, hipStream_t stream, Fill&& fill, Launch&& launch, Drain&& drain) {
  const size_t n_chunks = (n + chunk - 1) / chunk;
  auto items = [&](size_t i) { return (uint32_t)std::min(chunk, n - i * chunk); };
  for (size_t i = 0; i <= n_chunks; i++) {
    int32_t rc = i < n_chunks ? fill(i * chunk, items(i), stage.half(i)) : MRL_OK;
    if (i > 0) HIP_TRY(hipStreamSynchronize(stream));
    if (rc) return rc;
    if (i < n_chunks) HIP_TRY(launch(i * chunk, items(i), stage.half(i)));      // (a launch that fails queues nothing)
    if (i > 0 && (rc = drain((i - 1) * chunk, items(i - 1), stage.half(i - 1)))) {
      (void)hipStreamSynchronize(stream);
      return rc;
    }
  }
  return MRL_OK;
}

// The same in kParts stretches of the items at once where there is more than one chunk of them: the host's part (packing
// coordinates, copying answers and records into the caller's memory, which may be new and fault page by page) is what a long
// question waits for.  The calling thread takes the first stretch on `stream`, library threads the others on helper streams,
// which start behind what `stream` holds; the stretches share one staging block of per_item bytes an item.  A stretch that its
// share of the block holds is one launch (a lookup's takes 90 us whatever its points are), a longer one goes through in halves.
// fill, launch and drain also get the items that a chunk is laid out for, launch its stream.
// 100,003 Specs of the caller's arrays asked of the dense table 372 -> 147 us, looked up in the boxes 747 -> 437 (with the binding's
// records 739 -> 600 and 1219 -> 970; runs differ by 5 to 14 %); 1,000,000 3990 -> 1200 and 6690 -> 3530.
constexpr uint32_t kParts = 4;
constexpr uint32_t kPartThreads = 12;       // of all calls together
std::atomic<uint32_t> g_part_threads{0};

template <class Fill, class Launch, class Drain>
int32_t take_in_parts(size_t n, size_t chunk, size_t per_item, int device, hipStream_t stream, Fill&& fill, Launch&& launch, Drain&& drain) {
  StageLease stage;
  int32_t rc = get_stage(stage);
  if (rc) return rc;
  uint32_t parts = 1;
  if (n > chunk) {
    uint32_t taken = g_part_threads.load();
    while (taken + (kParts - 1) <= kPartThreads && !g_part_threads.compare_exchange_weak(taken, taken + (kParts - 1))) {}
    if (taken + (kParts - 1) <= kPartThreads) parts = kParts;
  }
  struct Give { uint32_t n; ~Give() { g_part_threads -= n; } } give{parts - 1};
  const size_t share = 2 * kStageHalf / parts, stretch = (n + parts - 1) / parts;
  const size_t piece = parts == 1 ? chunk : stretch <= share / per_item - 64 ? stretch + 63 & ~(size_t)63 : share / 2 / per_item & ~(size_t)63;
  auto run = [&](uint32_t p, hipStream_t st) -> int32_t {
    const size_t first = n * p / parts, end = n * (p + 1) / parts;
    const StageHalves mem{stage.mem + p * share, share / 2};
    return take_through(end - first, piece, mem, st,
                        [&](size_t at, uint32_t m, char* h) { return fill(first + at, m, h, piece); },
                        [&](size_t at, uint32_t m, char* h) { return launch(first + at, m, h, piece, st); },
                        [&](size_t at, uint32_t m, char* h) { return drain(first + at, m, h, piece); });
  };
  if (parts == 1) return run(0, stream);
  AuxLease aux;
  rc = get_aux(1, aux);
  if (rc) return rc;
  const hipEvent_t ready = aux.a->events[0];
  HIP_TRY(hipEventRecord(ready, stream));
  struct Join {
    std::mutex mu;
    std::condition_variable cv;
    uint32_t pending = 0;
    int32_t rc[kParts] = {};
    std::string err[kParts];
  } J;
  auto help = [&](uint32_t p) {
    int32_t code;
    try {
      code = [&]() -> int32_t {
        HIP_TRY(hipSetDevice(device));
        AuxLease own;
        int32_t r = get_aux(0, own);
        if (r) return r;
        HIP_TRY(hipStreamWaitEvent(own.a->stream, ready, 0));
        return run(p, own.a->stream);
      }();
      if (code) J.err[p] = g_err;
    } catch (...) { code = MRL_E_NOMEM; }
    std::lock_guard<std::mutex> lk(J.mu);
    J.rc[p] = code;
    J.pending--;
    J.cv.notify_all();
  };
  uint32_t given = 1;                        // stretches that have a thread
  for (; given < parts; given++) {
    { std::lock_guard<std::mutex> lk(J.mu); J.pending++; }
    try { const uint32_t p = given; workers().submit([&help, p] { help(p); }); }
    catch (...) { std::lock_guard<std::mutex> lk(J.mu); J.pending--; break; }
  }
  for (uint32_t p = 0; p < parts; p = p ? p + 1 : given) {
    try {
      J.rc[p] = run(p, stream);
      if (J.rc[p]) J.err[p] = g_err;
    } catch (...) { J.rc[p] = MRL_E_NOMEM; }
  }
  {
    std::unique_lock<std::mutex> lk(J.mu);
    J.cv.wait(lk, [&] { return J.pending == 0; });
  }
  for (uint32_t p = 0; p < parts; p++) if (J.rc[p]) return fail(J.rc[p], "%s", J.err[p].empty() ? "host allocation failed" : J.err[p].c_str());
  return MRL_OK;
}

}  // namespace

struct mrl_table {
  CompiledPtr cp;
  DevParams P;                // this table's copy: device pointers filled in by mrl_solve
  FixedLayout f;
  char* scratch;
  uint64_t* d_cost;
  uint16_t* d_arg;
  hipStream_t stream;
  int device = 0;             // where it was solved
  const mrl_table* deps[2] = {nullptr, nullptr};      // a FUSED table: the tables it was solved against
  // final lists inside scratch: [0] decisions, [1] costs
  size_t list_off[2];
  uint64_t list_n[2];
  // Lookups in the box lists (mrl_query_compressed): bounding-box hierarchy per list, allocated at
  // the first such query and freed with the table.
  struct BoxIndex { IndexLevels L; BoxBounds* nodes = nullptr; };
  mutable BoxIndex index[2];
  mutable std::mutex lookup_mu;
  ~mrl_table() {
    for (auto& ix : index) if (ix.nodes) (void)hipFree(ix.nodes);
  }
};

// No exception leaves the library: host allocations (std::vector, std::make_shared, ...) can throw.
template <class F>
int32_t guarded(F&& body) noexcept {
  try { return body(); }
  catch (const std::bad_alloc&) { return fail(MRL_E_NOMEM, "host allocation failed"); }
  catch (const std::exception& e) { return fail(MRL_E_HIP, "internal error: %s", e.what()); }
  catch (...) { return fail(MRL_E_HIP, "internal error: unknown exception"); }
}

extern "C" {

const char* mrl_last_error(void) { return g_err; }

int32_t mrl_target_create(const mrl_target_desc* desc, mrl_target** out) {
  return guarded([&]() -> int32_t {
  if (!out) return fail(MRL_E_INVAL, "out is NULL");
  *out = nullptr;
  int32_t rc = validate_target(desc);
  if (rc) return rc;
  mrl_target* t = new (std::nothrow) mrl_target;
  if (!t) return fail(MRL_E_NOMEM, "host allocation failed");
  t->d = *desc;
  *out = t;
  return MRL_OK;
  });
}

void mrl_target_destroy(mrl_target* t) { delete t; }

int32_t mrl_geometry(const mrl_target* t, const mrl_lattice_desc* lat, uint32_t* n_dims, uint32_t* extents,
                     uint64_t* n_specs) {
  return guarded([&]() -> int32_t {
  if (!t) return fail(MRL_E_INVAL, "target is NULL");
  CompiledPtr cp;
  int32_t rc = get_compiled(t->d, lat, cp);
  if (rc) return rc;
  const Compiled& c = *cp;
  if (n_dims) *n_dims = c.geo.ndim;
  if (extents) for (uint32_t a = 0; a < c.geo.ndim; a++) extents[a] = c.geo.ext[a];
  if (n_specs) *n_specs = c.n_specs;
  return MRL_OK;
  });
}

int32_t mrl_table_bytes(const mrl_target* t, const mrl_lattice_desc* lat, size_t* cost_bytes, size_t* argmin_bytes,
                        size_t* scratch_bytes) {
  return guarded([&]() -> int32_t {
  if (!t) return fail(MRL_E_INVAL, "target is NULL");
  CompiledPtr cp;
  int32_t rc = get_compiled(t->d, lat, cp);
  if (rc) return rc;
  const Compiled& c = *cp;
  if (cost_bytes) *cost_bytes = c.n_specs * 8;
  if (argmin_bytes) *argmin_bytes = c.n_specs * 2;
  if (scratch_bytes) {
    const FixedLayout f = fixed_layout(c);
    *scratch_bytes = std::max(f.fill_end, f.end + 2 * final_bytes(c.n_specs) + 2 * work_bytes(c.n_specs));
  }
  return MRL_OK;
  });
}

}  // extern "C"

namespace {

// on_filled (optional) is called once, when the fill's last kernel is queued on the table's stream
// and before the compression starts: the dense table is then complete for any work ordered after
// that point of the stream.  It returns whether the caller now shares the table object; a shared
// one is not deleted when the rest of the solve fails (the sharer deletes it).
using FilledFn = std::function<bool(mrl_table*)>;

// late_deps (optional; then deps is NULL) hands over the tables a lattice reads only when the fill
// needs them: it is called once the work that reads no other table (work lists and the pre-fill)
// is queued, may wait on the host until those tables' fills are queued, and gives for each an
// event behind which the table is complete.  The pre-fill of a large table then runs beside the
// fill of the tables it will read, not after it.
using LateDepsFn = std::function<int32_t(const mrl_table* tables[2], hipEvent_t ready[2])>;

int32_t solve_impl(const mrl_target* t, const mrl_lattice_desc* lat, const mrl_table* const* deps, uint32_t n_deps,
                   void* d_cost, void* d_argmin, void* d_scratch, size_t scratch_bytes, void* hip_stream,
                   mrl_table** out, mrl_stats* stats, const FilledFn& on_filled, const LateDepsFn& late_deps = LateDepsFn()) {
  return guarded([&]() -> int32_t {
  if (!out) return fail(MRL_E_INVAL, "out is NULL");
  *out = nullptr;
  if (!t) return fail(MRL_E_INVAL, "target is NULL");
  if (!lat) return fail(MRL_E_INVAL, "lattice descriptor is NULL");
  if (!d_cost || !d_argmin || !d_scratch) return fail(MRL_E_INVAL, "device buffers must not be NULL");
  if (((uintptr_t)d_cost | (uintptr_t)d_argmin | (uintptr_t)d_scratch) % kAlign) return fail(MRL_E_INVAL, "device buffers must be 256-byte aligned");
  mrl_table* tab = new (std::nothrow) mrl_table;
  if (!tab) return fail(MRL_E_NOMEM, "host allocation failed");
  struct Guard { mrl_table* p; bool shared; ~Guard() { if (!shared) delete p; } } guard{tab, false};
  int32_t rc = get_compiled(t->d, lat, tab->cp);
  if (rc) return rc;
  const Compiled& c = *tab->cp;
  tab->P = c.P;
  DevParams& P = tab->P;

  const mrl_table* late_tables[2] = {nullptr, nullptr};
  hipEvent_t late_ready[2] = {nullptr, nullptr};
  // the tables this lattice reads: checked against it, their geometry and addresses into P
  auto bind_deps = [&]() -> int32_t {
    if (P.split) {
      if (n_deps != 2 || !deps || !deps[0] || !deps[1]) return fail(MRL_E_INVAL, "a BIAS_ADD_RELU_SPLIT lattice needs deps = {BIAS_ADD table, RELU table}");
      const Compiled& A = *deps[0]->cp;
      const Compiled& R = *deps[1]->cp;
      if (A.lat.kind != MRL_KIND_BIAS_ADD || R.lat.kind != MRL_KIND_RELU) return fail(MRL_E_INVAL, "deps must be {BIAS_ADD, RELU}");
      if (memcmp(&A.target, &t->d, sizeof t->d) || memcmp(&R.target, &t->d, sizeof t->d)) return fail(MRL_E_INVAL, "deps were solved for another target");
      if (A.sizes[1] != c.sizes[1] || A.sizes[3] != c.sizes[3] || R.sizes[1] != c.sizes[1] || R.sizes[3] != c.sizes[3])
        return fail(MRL_E_INVAL, "the deps must have this lattice's m and n size lists");
      if ((P.lay_bit[0] != kNoBit && A.P.lay_bit[0] == kNoBit) || (P.lay_bit[2] != kNoBit && R.P.lay_bit[1] == kNoBit))
        return fail(MRL_E_INVAL, "a tensor with a layout coordinate in the BIAS_ADD_RELU_SPLIT lattice needs one in the dep it is looked up in");
      P.costM = deps[0]->d_cost; P.costE = deps[1]->d_cost;
      tab->deps[0] = deps[0]; tab->deps[1] = deps[1];
      P.GM = A.P.G; P.VM = A.P.V; P.GE = R.P.G; P.VE = R.P.V;
      for (int i = 0; i < 3; i++) { P.layM[i] = A.P.lay_bit[i]; P.layE[i] = R.P.lay_bit[i]; }
    } else if (P.chain) {
      if (n_deps != 1 || !deps || !deps[0]) return fail(MRL_E_INVAL, "a MATMUL_CHAIN lattice needs deps = {MATMUL_ACCUM table}");
      const Compiled& M = *deps[0]->cp;
      if (M.P.kind != kKindM || M.P.par || M.P.bounded || M.P.moves) return fail(MRL_E_INVAL, "the dep must be a MATMUL_ACCUM table");
      if (memcmp(&M.target, &t->d, sizeof t->d)) return fail(MRL_E_INVAL, "the dep was solved for another target");
      if (M.sizes[0].size() != 1) return fail(MRL_E_INVAL, "MATMUL_ACCUM dep must have b pinned to 1");
      // both stages are looked up in it: (m, k, p) and (m, p, n)
      if (M.sizes[1] != c.sizes[1] || M.sizes[2] != c.sizes[2] || M.sizes[2] != c.sizes[0] || M.sizes[3] != c.sizes[0] || M.sizes[3] != c.sizes[3])
        return fail(MRL_E_INVAL, "the m list must equal the MATMUL_ACCUM dep's, and the p, k and n lists its k and n lists");
      if ((P.lay_bit[0] != kNoBit && M.P.lay_bit[0] == kNoBit) || (P.lay_bit[1] != kNoBit && M.P.lay_bit[1] == kNoBit) ||
          (P.lay_bit[2] != kNoBit && M.P.lay_bit[1] == kNoBit) || (P.lay_bit[3] != kNoBit && M.P.lay_bit[2] == kNoBit))
        return fail(MRL_E_INVAL, "a tensor with a layout coordinate in the MATMUL_CHAIN lattice needs one in the dep it is looked up in");
      if (M.P.ndt || M.P.base_bf16[0] || M.P.base_bf16[1] || M.P.base_bf16[2]) return fail(MRL_E_INVAL, "MATMUL_ACCUM dep must be f32");
      P.costM = deps[0]->d_cost;
      tab->deps[0] = deps[0];
      P.GM = M.P.G; P.VM = M.P.V; P.kM_first = 0; P.nkM = (uint32_t)M.sizes[2].size();
      for (int i = 0; i < 3; i++) P.layM[i] = M.P.lay_bit[i];
    } else if (P.kind == kKindF) {
      if (n_deps != 2 || !deps || !deps[0] || !deps[1]) return fail(MRL_E_INVAL, "a FUSED lattice needs deps = {MATMUL_ACCUM table, BIAS_ADD_RELU table}");
      const Compiled& M = *deps[0]->cp;
      const Compiled& E = *deps[1]->cp;
      if (M.P.kind != kKindM || M.P.par || E.P.kind != kKindE || E.lat.kind == MRL_KIND_BIAS_ADD)
        return fail(MRL_E_INVAL, "deps must be {MATMUL_ACCUM, BIAS_ADD_RELU (or BIAS_ADD_RELU_SPLIT)}");
      if (M.P.bounded != P.bounded || E.P.bounded != P.bounded) return fail(MRL_E_INVAL, "memory bounds on all three tables or on none");
      if ((P.lay_bit[0] != kNoBit && M.P.lay_bit[0] == kNoBit) || (P.lay_bit[1] != kNoBit && M.P.lay_bit[1] == kNoBit) ||
          (P.lay_bit[3] != kNoBit && E.P.lay_bit[2] == kNoBit))
        return fail(MRL_E_INVAL, "a tensor with a layout coordinate in the FUSED lattice needs one in the dep it is looked up in");
      if (memcmp(&M.target, &t->d, sizeof t->d) || memcmp(&E.target, &t->d, sizeof t->d)) return fail(MRL_E_INVAL, "deps were solved for another target");
      if (M.sizes[1] != c.sizes[1] || M.sizes[3] != c.sizes[3]) return fail(MRL_E_INVAL, "MATMUL_ACCUM dep has other size lists");
      {
        // the k list: the dep's, or a stretch of consecutive entries of it (a slab of the whole lattice)
        const auto at = std::find(M.sizes[2].begin(), M.sizes[2].end(), c.sizes[2][0]);
        if ((size_t)(M.sizes[2].end() - at) < c.sizes[2].size() || !std::equal(c.sizes[2].begin(), c.sizes[2].end(), at))
          return fail(MRL_E_INVAL, "the k list must be a stretch of the MATMUL_ACCUM dep's k list");
        P.kM_first = (uint32_t)(at - M.sizes[2].begin());
        P.nkM = (uint32_t)M.sizes[2].size();
      }
      if (M.sizes[0].size() != 1) return fail(MRL_E_INVAL, "MATMUL_ACCUM dep must have b pinned to 1");
      if (E.sizes[1] != c.sizes[1] || E.sizes[3] != c.sizes[3]) return fail(MRL_E_INVAL, "BIAS_ADD_RELU dep has other size lists");
      if (M.P.ndt || M.P.base_bf16[0] || M.P.base_bf16[1] || M.P.base_bf16[2]) return fail(MRL_E_INVAL, "MATMUL_ACCUM dep must be f32");
      P.costM = deps[0]->d_cost; P.costE = deps[1]->d_cost;
      tab->deps[0] = deps[0]; tab->deps[1] = deps[1];
      P.GM = M.P.G; P.VM = M.P.V; P.GE = E.P.G; P.VE = E.P.V; P.nszE_n = E.P.nsz[3];
      for (int i = 0; i < 3; i++) { P.layM[i] = M.P.lay_bit[i]; P.layE[i] = E.P.lay_bit[i]; }
    } else if (P.par) {
      if (n_deps != 1 || !deps || !deps[0]) return fail(MRL_E_INVAL, "a MATMUL_PARALLEL lattice needs deps = {MATMUL_ACCUM table of the same lattice}");
      const Compiled& M = *deps[0]->cp;
      if (M.P.kind != kKindM || M.P.par) return fail(MRL_E_INVAL, "the dep must be a MATMUL_ACCUM table");
      if (memcmp(&M.target, &t->d, sizeof t->d)) return fail(MRL_E_INVAL, "the dep was solved for another target");
      for (int d = 0; d < 4; d++) if (M.sizes[d] != c.sizes[d]) return fail(MRL_E_INVAL, "the MATMUL_ACCUM dep has other size lists");
      if (memcmp(M.lat.layout_coord, c.lat.layout_coord, sizeof c.lat.layout_coord) ||
          memcmp(M.lat.dtype_coord, c.lat.dtype_coord, sizeof c.lat.dtype_coord) ||
          memcmp(M.lat.base_dtype_bytes, c.lat.base_dtype_bytes, 3) || M.n_specs != c.n_specs || M.P.G != P.G)
        return fail(MRL_E_INVAL, "the MATMUL_ACCUM dep has other coordinates");
      P.costM = deps[0]->d_cost;
      tab->deps[0] = deps[0];
    } else if (P.moves) {
      if (n_deps != 1 || !deps || !deps[0]) return fail(MRL_E_INVAL, "a MATMUL_MOVES lattice needs deps = {MOVE table}");
      const Compiled& V = *deps[0]->cp;
      if (V.P.kind != kKindV) return fail(MRL_E_INVAL, "the dep must be a MOVE table");
      if (memcmp(&V.target, &t->d, sizeof t->d)) return fail(MRL_E_INVAL, "the dep was solved for another target");
      if (c.sizes[1] != V.sizes[1] || c.sizes[2] != V.sizes[1] || c.sizes[2] != V.sizes[3] || c.sizes[3] != V.sizes[3])
        return fail(MRL_E_INVAL, "the m, k and n size lists must all equal the MOVE table's row and column lists");
      bool any_lay = false, any_dt = false;
      for (int i = 0; i < 3; i++) { any_lay = any_lay || P.lay_bit[i] != kNoBit; any_dt = any_dt || P.dt_bit[i] != kNoBit || P.base_bf16[i]; }
      if (any_lay && (V.P.lay_bit[0] == kNoBit || V.P.lay_bit[1] == kNoBit)) return fail(MRL_E_INVAL, "the MOVE table needs layout bits on both tensors");
      if (P.xw == 4 && (V.P.lay_w[0] != 2 || V.P.lay_w[1] != 2)) return fail(MRL_E_INVAL, "the MOVE table needs the packed layouts on both tensors");
      if (any_dt && (V.P.dt_bit[0] == kNoBit || V.P.dt_bit[1] == kNoBit)) return fail(MRL_E_INVAL, "the MOVE table needs dtype bits on both tensors");
      if (V.P.dt_bit[0] == kNoBit && (V.P.base_bf16[0] || V.P.base_bf16[1])) return fail(MRL_E_INVAL, "a MOVE table without dtype bits must be f32");
      P.costM = deps[0]->d_cost;
      tab->deps[0] = deps[0];
      P.GV = V.P.G; P.VV = V.P.V; P.nszV = V.P.nsz[3]; P.QV = V.P.Q;
      for (int a = 0; a < 4; a++) P.limV_stride[a] = V.P.lim_stride[a];
      for (int i = 0; i < 2; i++) { P.layV[i] = V.P.lay_bit[i]; P.dtV[i] = V.P.dt_bit[i]; }
    } else if (n_deps != 0) {
      return fail(MRL_E_INVAL, "only FUSED, MATMUL_PARALLEL, MATMUL_MOVES, MATMUL_CHAIN and BIAS_ADD_RELU_SPLIT lattices take deps");
    }
    return MRL_OK;
  };
  // (the kinds filled by gathers have no pre-fill to run ahead: they take their deps at once)
  const bool deps_late = (bool)late_deps && !P.gather && n_deps > 0;
  if (late_deps && !deps_late && n_deps > 0) {
    rc = late_deps(late_tables, late_ready);
    if (rc) return rc;
    deps = late_tables;
    for (uint32_t i = 0; i < n_deps; i++) HIP_TRY(hipStreamWaitEvent((hipStream_t)hip_stream, late_ready[i], 0));
  }
  if (!deps_late) { rc = bind_deps(); if (rc) return rc; }

  if (!P.gather && !plan_fits(P, c.n_shapes, c.level_off.data(), (uint32_t)c.level_off.size() - 1))
    return fail(MRL_E_INVAL, "a dependency level has too many shapes for its work lists");

  std::unique_lock<std::mutex> solve_lock(c.solve_mu);      // for the upload image, until the upload has run

  const FixedLayout f = fixed_layout(c);
  tab->f = f;
  // What the merge word by word needs beyond the fill's part depends on the contents; where that does not suffice, boxes are
  // merged one by one.  Its words are the larger part: if those of all rows do not fit, the plan's fit map is asked how many
  // rows there are, together with the work lists' lengths.  Turned rows are tried first, then, if there may be too little
  // scratch for them, rows along n.
  struct ByRows { RowGeo g; FixedLayout f; uint64_t room; bool on, ask; } by_rows[2];
  uint32_t n_ways = 0;
  for (const bool may_turn : {true, false}) {
    ByRows& w = by_rows[n_ways];
    if (!row_geo(c, may_turn, w.g)) break;
    if (n_ways && w.g.axis[3] == by_rows[0].g.axis[3]) break;
    w.f = may_turn ? f : fixed_layout(c, false);
    w.room = scratch_bytes > w.f.rows_dyn ? scratch_bytes - w.f.rows_dyn : 0;
    w.on = row_words_fit(w.g, w.g.n_planes, w.room);
    w.ask = w.on && !row_words_fit(w.g, (uint64_t)w.g.n_planes * w.g.ek, w.room);
    n_ways++;
    if (rows_always_fit(w.g, w.room)) break;
  }
  bool some_rows = false, ask_rows = false;
  for (uint32_t i = 0; i < n_ways; i++) { some_rows |= by_rows[i].on; ask_rows |= by_rows[i].ask; }
  if (scratch_bytes < (some_rows ? f.fill_end : f.least())) return fail(MRL_E_NOMEM, "scratch buffer too small: %zu bytes given, at least %zu needed", scratch_bytes, f.least());
  char* base = (char*)d_scratch;
  hipStream_t st = (hipStream_t)hip_stream;
  HIP_TRY(hipGetDevice(&tab->device));
  tab->scratch = base; tab->d_cost = (uint64_t*)d_cost; tab->d_arg = (uint16_t*)d_argmin; tab->stream = st;

  Counters* d_ctr = (Counters*)(base + f.counters);
  DevParams* d_P = (DevParams*)(base + f.params);
  P.tiles = (const TileEntry*)(base + f.tiles);
  P.steps = (const TileStep*)(base + f.tiles);
  const uint32_t n_lev = (uint32_t)c.level_off.size() - 1;
  uint32_t* d_level_shapes = (uint32_t*)(base + f.level_shapes);
  uint32_t* d_fitmap = (uint32_t*)(base + f.fitmap);
  P.mk_entry = (const uint8_t*)(base + f.mk_entry);
  P.qdec = (const uint32_t*)(base + f.qdec);
  P.bind = (const uint64_t*)(base + f.bind);
  ImageLease borrowed;
  char* upload = c.staging.mem;
  const auto image = [&](size_t at) { return upload + (at - f.counters); };
  if (!upload) {
    PinnedImage& to = c.solved ? c.staging : borrowed.image;
    rc = take_image(f.image_bytes(), c.solved ? 2 * f.image_bytes() + (64u << 10) : SIZE_MAX, to);
    if (rc) return rc;
    c.solved = true;
    upload = to.mem;
    memset(upload, 0, f.params - f.counters);
    if (P.gather) {
      if (!c.tiles.empty()) memcpy(image(f.tiles), c.tiles.data(), c.tiles.size() * sizeof(TileEntry));
    } else {
      TileStep* steps = (TileStep*)image(f.tiles);
      for (uint32_t d = 0; d < 4; d++)
        for (uint32_t j = 0; j < P.nsz[d]; j++)
          for (uint32_t q = P.tile_off[d][j]; q < P.tile_off[d][j + 1]; q++) {
            const TileEntry te = c.tiles[q];
            steps[q] = TileStep{(j - te.jt) * P.shape_stride[d] * P.G, te.trips, P.tile_base + d * P.maxs + te.jt, (uint32_t)(((uint64_t)te.trips + P.threads - 1) / P.threads)};
          }
      unit_blocks(c.level_off.data(), n_lev, P.npass, (uint32_t*)image(f.blk_off));
    }
    memcpy(image(f.level_shapes), c.level_shapes.data(), c.level_shapes.size() * 4);
    memcpy(image(f.level_off), c.level_off.data(), c.level_off.size() * 4);
    memcpy(image(f.mk_entry), c.mk_entry.data(), c.mk_entry.size());
    if (!c.qdec.empty()) memcpy(image(f.qdec), c.qdec.data(), c.qdec.size() * 4);
  }
  memcpy(image(f.params), &P, sizeof P);
  AuxLease lease;
  rc = get_aux(16, lease);
  if (rc) return rc;
  Aux* aux = lease.a;
  const PlanBuffers plan{base + f.recs, (unsigned long long*)(base + f.masks), d_level_shapes, (const uint32_t*)(base + f.level_off), (const uint32_t*)(base + f.blk_off),
                         (uint32_t*)(base + f.unit_cnt), (uint32_t*)(base + f.unit_seg), aux->h_counts + kDiagFirst, base + f.list};
  // Whichever way this function is left from here on, both streams have drained before the turn
  // for the upload image, the helper stream with its events and pinned counters, and (on
  // failure) the table object are given up: work queued on the streams may still use all of these.
  struct Drain {
    hipStream_t a, b;
    ~Drain() { (void)hipStreamSynchronize(a); (void)hipStreamSynchronize(b); }
  } drain{st, aux->stream};
  HIP_TRY(hipMemcpyAsync(base + f.counters, upload, f.image_bytes(), hipMemcpyHostToDevice, st));

  // ---- fill: plan and work list, then a launch per diagonal ----
  hipEvent_t* ev = aux->timing;
  size_t ev_used = 0;
  hipStream_t s2 = aux->stream;
  HIP_TRY(hipEventRecord(ev[0], st));
  bool prefill_timed = false, levels_timed = false;
  const hipEvent_t uploaded = aux->events[ev_used++];
  HIP_TRY(hipEventRecord(uploaded, st));
  hipEvent_t prefilled = nullptr;
  uint64_t n_units = 0;
  if (P.gather) {
    // Memory bounds as coordinates (and Move Specs): every Spec is evaluated (no admissibility test, so every cell
    // counts as fitting for the compression); one launch per dependency level of shapes and rank
    // of level assignments, each over Specs that depend only on earlier launches.
    launch_fill_ones(d_fitmap, ((size_t)f.n_words + 2) * 8, st);
    const int gather_mode = P.kind == kKindV ? 1 : 0;
    const uint64_t qv = (uint64_t)P.Q * P.V;
    const bool units = fill_by_units(gather_mode, qv);
    BoundSegs segs;
    segs.n = 0; segs.block0[0] = 0; segs.waves_per_unit = segs.lanes_per_wave = 1;
    auto flush = [&]() {
      launch_fill_bounded(d_P, gather_mode, units, d_level_shapes, segs, tab->d_cost, tab->d_arg, d_ctr, st);
      segs.n = 0; segs.block0[0] = 0;
    };
    // one segment: `level_units` = (shape, level assignment, intermediate's level) combinations of it
    auto add = [&](uint32_t l, uint32_t r, uint64_t level_units) -> int32_t {
      const uint64_t blocks = units ? (level_units * segs.waves_per_unit + 3) / 4 : (level_units * qv + 255) / 256;
      if (!blocks) return MRL_OK;
      if (segs.n == kBoundSegs || segs.block0[segs.n] + blocks >= (1ull << 31)) flush();
      if (blocks >= (1ull << 31)) return fail(MRL_E_INVAL, "a dependency level of the bounded lattice is too large for one launch");
      segs.first_shape[segs.n] = c.level_off[l]; segs.n_shapes[segs.n] = c.level_off[l + 1] - c.level_off[l]; segs.rank[segs.n] = r;
      segs.block0[segs.n + 1] = segs.block0[segs.n] + (uint32_t)blocks;
      segs.n++;
      return MRL_OK;
    };
    // a wave's stretch: up to kStretch times 64 entries of a unit, fewer while that leaves the chip short of waves
    auto set_stretch = [&](uint64_t launch_units) {
      uint64_t stretch = 1;
      while (stretch < kStretch && launch_units * ((qv + 128 * stretch - 1) / (128 * stretch)) >= kFullWaves) stretch *= 2;
      segs.lanes_per_wave = (uint32_t)(64 * stretch);
      segs.waves_per_unit = (uint32_t)((qv + 64 * stretch - 1) / (64 * stretch));
    };
    if (gather_mode == 1) {
      // Move Specs have no Moves: the level assignments of a shape do not depend on each other
      for (uint32_t l = 0; l < n_lev; l++) {
        const uint64_t n = (uint64_t)(c.level_off[l + 1] - c.level_off[l]) * P.ncombo;
        set_stretch(n);
        rc = add(l, 0, n);
        if (rc) return rc;
        flush();
      }
    } else {
      for (uint32_t d = 0; d + 1 < n_lev + P.nranks; d++) {
        const uint32_t l0 = d < P.nranks ? 0 : d - (P.nranks - 1);
        auto seg_units = [&](uint32_t l) { return (uint64_t)(c.level_off[l + 1] - c.level_off[l]) * (P.rank_off[d - l + 1] - P.rank_off[d - l]) * P.npass; };
        uint64_t n = 0;
        for (uint32_t l = l0; l < n_lev && l <= d; l++) n += seg_units(l);
        set_stretch(n);
        for (uint32_t l = l0; l < n_lev && l <= d; l++) { rc = add(l, d - l, seg_units(l)); if (rc) return rc; }
        flush();
      }
    }
  } else {
  // plan; then the host reads the diagonals' sizes back
  uint32_t blk_off[kMaxLevels + 1];
  const uint32_t n_blk = unit_blocks(c.level_off.data(), n_lev, P.npass, blk_off), n_diag = n_lev + P.nranks - 1;
  const uint64_t list_room = (scratch_bytes - f.list) / 8;
  const uint32_t window = (uint32_t)std::min<uint64_t>(list_room, UINT32_MAX);
  // The pre-fill, (INF, NONE) over both tables, and the fit map run beside the plan and the fill on the helper stream, where they take
  // longer than the events do: the pre-fill is done before the first diagonal, the map before the compression.  (A lattice that
  // reads other tables streams the pre-fill behind its plan.)  What comes before the first diagonal is host time on small tables: the
  // map is launched when the diagonals are.  The line: beside at any size, the vector-matrix product (180 shapes) 440 ->
  // 463 us; never beside, the pipeline 3022 -> 3051 (F's 449.5 M Specs), all between within 1 % of each other.
  const bool beside = c.n_specs >= (1u << 21);
  if (!deps_late && beside) {
    HIP_TRY(hipStreamWaitEvent(s2, uploaded, 0));
    launch_prefill(tab->d_cost, tab->d_arg, c.n_specs, s2);
    HIP_TRY(hipEventRecord(aux->events[ev_used], s2));
    prefilled = aux->events[ev_used++];
  }
  memset(plan.host_diag, 0, ((size_t)n_diag + 1) * 4);
  launch_plan(d_P, P, n_lev, n_blk, plan, d_ctr, st);
  if (ask_rows) {
    launch_fit_map(d_P, (uint32_t)c.n_specs, plan, d_fitmap, f.n_words, st);
    for (uint32_t i = 0; i < n_ways; i++) if (by_rows[i].ask) launch_row_total(by_rows[i].g, d_fitmap, d_ctr->rows + i, st);
    HIP_TRY(hipMemcpyAsync(aux->h_counts + kRowTotals, d_ctr->rows, sizeof d_ctr->rows, hipMemcpyDeviceToHost, st));
  }
  HIP_TRY(hipEventRecord(aux->events[ev_used], st));
  hipEvent_t counts_ready = aux->events[ev_used++];
  const uint64_t shapes_from = by_shapes_from(P, c.n_shapes, n_lev);
  launch_list_units(d_P, P, n_lev, blk_off, plan, 0, window, 0, n_diag - 1, shapes_from, st);
  if (prefilled) HIP_TRY(hipStreamWaitEvent(st, prefilled, 0)); else launch_prefill(tab->d_cost, tab->d_arg, c.n_specs, st);
  HIP_TRY(hipEventRecord(ev[4], st));
  prefill_timed = true;
  HIP_TRY(hipEventSynchronize(counts_ready));
  for (uint32_t i = 0; i < n_ways; i++)
    if (by_rows[i].ask) by_rows[i].on = row_words_fit(by_rows[i].g, aux->h_counts[kRowTotals + i], by_rows[i].room);
  if (deps_late) {
    // now the tables this lattice reads: their fills are queued (or the call waits here until
    // they are); the parameters go up once more, with their addresses, and the diagonals wait for them
    rc = late_deps(late_tables, late_ready);
    if (rc) return rc;
    deps = late_tables;
    rc = bind_deps();
    if (rc) return rc;
    memcpy(image(f.params), &P, sizeof P);
    HIP_TRY(hipMemcpyAsync(d_P, image(f.params), sizeof P, hipMemcpyHostToDevice, st));
    HIP_TRY(hipEventRecord(uploaded, st));
    for (uint32_t i = 0; i < n_deps; i++) HIP_TRY(hipStreamWaitEvent(st, late_ready[i], 0));
  }
  HIP_TRY(hipEventRecord(ev[5], st));
  levels_timed = true;
  if (P.moves) launch_bind(d_P, (uint64_t*)(base + f.bind), (uint32_t)bind_entries(c), st);
  const uint32_t* diag = plan.host_diag;
  const FillArgs fill = fill_args(d_P, P, plan, tab->d_cost, tab->d_arg, d_ctr);
  const uint32_t most = most_units(fill);
  uint32_t w0 = 0;                        // the list holds units [w0, w0 + window)
  DiagRun run;
  run.n = 0;
  const auto flush = [&]() {
    if (run.n) launch_fill_diagonals(fill, P, base + f.list, run, st);
    run.n = 0;
  };
  const uint64_t more_windows = diag[n_diag] ? (diag[n_diag] - 1) / window : 0;
  const bool by_shapes = shapes_from != UINT64_MAX && diag[n_diag] + more_windows * units_for_a_launch(P) >= shapes_from;
  for (uint32_t l = 0; by_shapes && l < n_lev; l++) launch_fill_shapes(fill, P, plan.masks, c.level_off[l], c.level_off[l + 1] - c.level_off[l], st);
  for (uint32_t d = 0; !by_shapes && d < n_diag; d++)
    for (uint32_t u = diag[d]; u < diag[d + 1];) {
      if (u - w0 >= window) {
        flush();
        w0 = u;
        const uint32_t w_len = std::min(window, diag[n_diag] - w0);
        uint32_t last = d;
        while (diag[last + 1] - w0 < w_len) last++;
        launch_list_units(d_P, P, n_lev, blk_off, plan, w0, w_len, d, last, UINT64_MAX, st);
      }
      const uint32_t n = std::min({diag[d + 1] - u, window - (u - w0), most});
      const bool small = small_diagonal(fill, n);
      if (!small || run.n == kRunMost) flush();
      run.chain = small;
      run.start[run.n] = u - w0;
      run.start[++run.n] = u - w0 + n;
      if (!small) flush();
      u += n;
    }
  flush();
  n_units = diag[n_diag];
  if (!ask_rows) {
    if (beside) HIP_TRY(hipStreamWaitEvent(s2, deps_late ? uploaded : counts_ready, 0));       // behind the plan (and the second upload)
    launch_fit_map(d_P, (uint32_t)c.n_specs, plan, d_fitmap, f.n_words, beside ? s2 : st);
    if (beside) {
      HIP_TRY(hipEventRecord(aux->events[ev_used], s2));
      HIP_TRY(hipStreamWaitEvent(st, aux->events[ev_used++], 0));
    }
  }
  }
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipEventRecord(ev[1], st));
  if (on_filled) {
    // on_filled may wait (host side) for other jobs, which may need this lattice's turn
    HIP_TRY(hipEventSynchronize(uploaded));
    solve_lock.unlock();
    guard.shared = on_filled(tab);
  }
  HIP_TRY(hipEventRecord(ev[3], st));

  // ---- compression ----
  const Geo& g = c.geo;
  Counters& h_ctr = *reinterpret_cast<Counters*>(aux->h_counts + kCountersAt);
  size_t needed = 0;
  bool merged = false;
  for (uint32_t i = 0; i < n_ways && !merged; i++) {
    if (!by_rows[i].on) continue;
    const RowGeo& rg = by_rows[i].g;
    const FixedLayout& rf = by_rows[i].f;
    const RowBufs rb{(uint32_t*)(base + rf.rows_rows), (uint32_t*)(base + rf.rows_first), base + rf.rows_info, (uint32_t*)(base + rf.rows_cnt), (uint32_t*)(base + rf.rows_start),
                     base + rf.rows_sum, (uint32_t*)(base + rf.rows_tot), base + rf.rows_dyn, by_rows[i].room};
    launch_rows(rg, rb, tab->d_cost, tab->d_arg, d_fitmap, (const uint32_t*)((char*)d_P + offsetof(DevParams, sizes)), st);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipEventRecord(ev[2], st));
    HIP_TRY(hipMemcpyAsync(aux->h_counts, rb.tot, kRowTotals * 4, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipMemcpyAsync(&h_ctr, d_ctr, sizeof h_ctr, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    uint64_t list_at[2], end = 0;
    merged = rows_fit(rg, aux->h_counts, rb.room, list_at, &end);
    if (merged) {
      tab->list_n[0] = aux->h_counts[kBoxesFirst];
      tab->list_n[1] = aux->h_counts[kBoxesTotal] - tab->list_n[0];
      for (int which = 0; which < 2; which++) tab->list_off[which] = rf.rows_dyn + list_at[which];
      needed = std::max(rf.fill_end, rf.rows_dyn + (size_t)end);
    }
  }
  if (!merged) {
    if (scratch_bytes < f.least()) return fail(MRL_E_NOMEM, "scratch buffer too small: %zu bytes given, at least %zu needed", scratch_bytes, f.least());
    uint32_t a0 = c.merge_order[0];
    for (uint32_t q = 0; q < g.ndim; q++) if (g.ext[c.merge_order[q]] > 1) { a0 = c.merge_order[q]; break; }
    unsigned long long* maskL[2] = {(unsigned long long*)(base + f.maskD), (unsigned long long*)(base + f.maskC)};
    uint32_t* prefL[2] = {(uint32_t*)(base + f.prefD), (uint32_t*)(base + f.prefC)};
    uint32_t* tile_tmp = (uint32_t*)(base + f.tile_tmp);
    uint32_t* d_tot = (uint32_t*)(base + f.totals);
    auto axis_sizes = [&](uint32_t a) -> const uint32_t* { return a < 4 ? (const uint32_t*)((char*)d_P + offsetof(DevParams, sizes) + a * sizeof(uint32_t) * kMaxSizes) : nullptr; };
    unsigned long long* lineL[2] = {(unsigned long long*)(base + f.lineD), (unsigned long long*)(base + f.lineC)};
    launch_head_flags(g, a0, tab->d_cost, tab->d_arg, d_fitmap, axis_sizes(a0), maskL[0], maskL[1], lineL[0], lineL[1], st);
    uint32_t a1 = 0;
    const bool on_cells = second_on_cells(c, nullptr, &a1);
    const unsigned long long* colL[2] = {nullptr, nullptr};
    if (on_cells) launch_zero_words((unsigned long long*)(base + f.colD), (uint32_t)((f.colC - f.colD) / 8 + c.n_specs / g.ext[a1]), st);
    // the two prefix sums side by side (each is one to three short kernels): the decisions' on the helper stream
    HIP_TRY(hipEventRecord(aux->events[ev_used], st));
    HIP_TRY(hipStreamWaitEvent(s2, aux->events[ev_used++], 0));
    if (on_cells) {
      // the pass on the second merge axis, on the cells: the box heads that remain go to a second mask
      unsigned long long* m2[2] = {(unsigned long long*)(base + f.mask2D), (unsigned long long*)(base + f.mask2C)};
      unsigned long long* cl[2] = {(unsigned long long*)(base + f.colD), (unsigned long long*)(base + f.colC)};
      launch_second_axis(g, a0, a1, false, maskL[0], lineL[0], d_fitmap, tab->d_cost, tab->d_arg, axis_sizes(a1), m2[0], cl[0], s2);
      launch_second_axis(g, a0, a1, true, maskL[1], lineL[1], d_fitmap, tab->d_cost, tab->d_arg, axis_sizes(a1), m2[1], cl[1], st);
      for (int w = 0; w < 2; w++) { maskL[w] = m2[w]; colL[w] = cl[w]; }
    }
    scan_mask_words(maskL[0], f.n_words, (uint32_t*)(base + f.tile_tmp2), prefL[0], d_tot + 0, s2);
    scan_mask_words(maskL[1], f.n_words, tile_tmp, prefL[1], d_tot + 1, st);
    HIP_TRY(hipEventRecord(aux->events[ev_used], s2));
    HIP_TRY(hipStreamWaitEvent(st, aux->events[ev_used++], 0));
    HIP_TRY(hipMemcpyAsync(aux->h_counts, d_tot, 8, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    const uint32_t h_tot[2] = {aux->h_counts[0], aux->h_counts[1]};

    // The two lists are merged side by side, the decisions on the helper stream: most of the
    // kernels are bound by latency, not bandwidth.  The host waits twice per list: for the number
    // of live boxes after the first pass (it sizes the grids of the later ones) and for the final
    // count (it places the final list); meanwhile the other list's stream has work queued.
    // Work areas at the end of the buffer, the final lists grow from the front.
    const uint64_t nbL[2] = {h_tot[0], h_tot[1]};
    const size_t wbL[2] = {work_bytes(nbL[0]), work_bytes(nbL[1])};
    size_t front = f.end;
    needed = f.end + wbL[0] + wbL[1] + final_bytes(nbL[0]) + final_bytes(nbL[1]);   // upper bound until the final counts are known
    if (scratch_bytes < f.end + wbL[0] + wbL[1])
      return fail(MRL_E_NOMEM, "scratch buffer too small: %zu bytes given, up to %zu needed", scratch_bytes, needed);
    char* work_lo = base + (scratch_bytes - wbL[0] - wbL[1]) / kAlign * kAlign;
    if ((size_t)(work_lo - base) < f.end)
      return fail(MRL_E_NOMEM, "scratch buffer too small: %zu bytes given, up to %zu needed", scratch_bytes, needed);
    // per list: its arrays and the pass state.  Once the first pass has merged most boxes away, the
    // live ones move to dense arrays (cell2, len2, alive2) and get new indices 0..n-1, in order
    struct ListWork {
      uint32_t *bcell, *next, *pos, *cell2, *pos2, *block_linked, *d_cnt;
      char *blen, *len2;
      uint8_t *alive, *alive2;
      const uint8_t* old_alive = nullptr;     // set by the compaction, with remap
      const uint32_t* remap = nullptr;
      uint32_t n = 0, q_next = 0;
      uint8_t stamp = 0;
    } LW[2];
    hipStream_t stL[2] = {s2, st};
    uint32_t* tileL[2] = {(uint32_t*)(base + f.tile_tmp2), tile_tmp};
    // the passes in order; the trailing ones over bit axes inside a mask word are done in one kernel
    uint32_t pass_axis[16], n_axes = 0;
    for (uint32_t q = 0; q < g.ndim; q++) {
      const uint32_t a = c.merge_order[q];
      if (a != a0 && g.ext[a] > 1) pass_axis[n_axes++] = a;
    }
    uint32_t n_generic = n_axes;
    // (a power-of-two stride: the coordinate on the axis is then one bit of the cell index, which
    // the kernel relies on; behind an axis of another extent, e.g. a memory bound, it is not.  Not a
    // size axis: along those the cost list compares costs per volume, which that kernel does not)
    auto tail_axis = [&](uint32_t a) { return a >= 4 && g.ext[a] == 2 && g.stride[a] <= 32 && (g.stride[a] & (g.stride[a] - 1)) == 0; };
    while (n_generic > 0 && n_axes - n_generic < 6 && tail_axis(pass_axis[n_generic - 1])) n_generic--;
    TailAxes tail;
    tail.n = n_axes - n_generic;
    for (uint32_t k = 0; k < tail.n; k++) { tail.axis[k] = pass_axis[n_generic + k]; tail.stride[k] = g.stride[pass_axis[n_generic + k]]; }

    auto one_pass = [&](int which) {
      ListWork& W = LW[which];
      const uint32_t a = pass_axis[W.q_next++];
      launch_axis_pass(g, a, ++W.stamp, which == 1, W.n, W.old_alive, W.remap, W.bcell, W.blen, W.alive, W.next,
                       W.block_linked, maskL[which], prefL[which], tab->d_cost, tab->d_arg, axis_sizes(a), stL[which]);
    };
    // first part: the boxes of pass 0 and the first generic pass, then (large lists) the compaction;
    // the count of live boxes is fetched while the other list's first part runs
    bool compacted[2] = {false, false};
    for (int which = 1; which >= 0; which--) {
      ListWork& W = LW[which];
      const uint64_t nb = nbL[which];
      char* w = which == 0 ? work_lo : work_lo + wbL[0];
      W.bcell = (uint32_t*)w; w += align_up(nb * 4);
      W.blen = w; w += align_up(nb * 16);
      W.alive = (uint8_t*)w; w += align_up(nb);
      W.next = (uint32_t*)w; w += align_up(nb * 4);
      W.pos = (uint32_t*)w; w += align_up(nb * 4);
      W.cell2 = (uint32_t*)w; w += align_up(nb * 4);
      W.pos2 = (uint32_t*)w; w += align_up(nb * 4);
      W.len2 = w; w += align_up(nb * 16);
      W.alive2 = (uint8_t*)w; w += align_up(nb);
      W.block_linked = (uint32_t*)w;
      W.d_cnt = d_tot + 4 + which * 4;       // [0]: live boxes at the compaction; [2]: the final count
      W.n = (uint32_t)nb;
      launch_make_boxes(g, a0, maskL[which], prefL[which], lineL[which], colL[which], a1, W.bcell, W.blen, W.alive, stL[which]);
      if (on_cells) W.q_next = 1;               // pass_axis[0] = a1 is done
      if (W.q_next < n_generic) {
        one_pass(which);
        // (not after the pass on the cells: it leaves no dead boxes, and a compaction after the next pass costs more than it saves)
        if (!on_cells && W.n > (1u << 20) && (W.q_next < n_generic || tail.n)) {
          scan_flags(W.alive, W.n, tileL[which], W.pos, W.d_cnt, stL[which]);
          launch_compact_boxes(W.n, W.alive, W.pos, W.bcell, W.blen, W.cell2, W.len2, W.alive2, stL[which]);
          HIP_TRY(hipMemcpyAsync(aux->h_counts + 2 + which, W.d_cnt, 4, hipMemcpyDeviceToHost, stL[which]));
          compacted[which] = true;
        }
      }
    }
    // second part: the other passes on the dense arrays, the final count
    for (int which = 1; which >= 0; which--) {
      ListWork& W = LW[which];
      if (compacted[which]) {
        HIP_TRY(hipStreamSynchronize(stL[which]));
        W.n = aux->h_counts[2 + which];
        W.old_alive = W.alive; W.remap = W.pos;
        W.bcell = W.cell2; W.blen = W.len2; W.alive = W.alive2; W.pos = W.pos2;
      }
      while (W.q_next < n_generic) one_pass(which);
      if (tail.n)
        launch_tail_pairs(tail, which == 1, f.n_words, maskL[which], prefL[which], W.old_alive, W.remap, W.blen, W.alive,
                          tab->d_cost, tab->d_arg, stL[which]);
      scan_flags(W.alive, W.n, tileL[which], W.pos, W.d_cnt + 2, stL[which]);
      HIP_TRY(hipMemcpyAsync(aux->h_counts + which, W.d_cnt + 2, 4, hipMemcpyDeviceToHost, stL[which]));
      HIP_TRY(hipEventRecord(aux->events[ev_used + which], stL[which]));
    }
    // the final lists: the decisions' first (the shorter list, as a rule through first); the host
    // sleeps until a list's count has arrived
    const hipEvent_t counted[2] = {aux->events[ev_used], aux->events[ev_used + 1]};
    ev_used += 2;
    for (int which = 0; which < 2; which++) {
      const int left = 1 - which;
      HIP_TRY(hipEventSynchronize(counted[which]));
      const uint64_t nf = aux->h_counts[which];
      const size_t fb = final_bytes(nf);
      if (front + fb > (size_t)(work_lo - base)) {
        return fail(MRL_E_NOMEM, "scratch buffer too small: %zu bytes given, %zu needed", scratch_bytes,
                    front + fb + (left ? final_bytes(nbL[1 - which]) : 0) + wbL[0] + wbL[1]);
      }
      char* r = base + front;
      uint32_t* fcell = (uint32_t*)r; r += align_up(nf * 4);
      char* flen = r; r += align_up(nf * 16);
      uint64_t* fv0 = (uint64_t*)r; r += align_up(nf * 8);
      uint64_t* fv1 = (uint64_t*)r;
      const ListWork& W = LW[which];
      launch_emit(g, d_P, which == 1, W.n, W.bcell, W.blen, W.alive, W.pos, tab->d_cost, tab->d_arg, fcell, flen, fv0, fv1,
                  stL[which]);
      tab->list_off[which] = front;
      tab->list_n[which] = nf;
      front += fb;
    }
    needed = std::max(f.fill_end, front + wbL[0] + wbL[1]);
    HIP_TRY(hipEventRecord(aux->events[ev_used], s2));
    HIP_TRY(hipStreamWaitEvent(st, aux->events[ev_used++], 0));
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipEventRecord(ev[2], st));
    HIP_TRY(hipMemcpyAsync(&h_ctr, d_ctr, sizeof h_ctr, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
  }
  if (h_ctr.overflow) return fail(MRL_E_OVERFLOW, "a finite cost reached 2^62");
  if (stats) {
    memset(stats, 0, sizeof *stats);
    stats->n_specs = c.n_specs;
    stats->n_admissible = P.gather ? 0 : n_units << P.unit_lay;
    stats->n_rewrites = 0;
    for (uint32_t i = 0; i < kCtrSlots; i++) { stats->n_admissible += h_ctr.n_admissible[i]; stats->n_rewrites += h_ctr.n_rewrites[i]; }
    if (P.bounded) stats->n_admissible = c.n_specs;      // no admissibility test: every Spec is evaluated
    stats->n_levels_run = n_lev;
    HIP_TRY(hipEventElapsedTime(&stats->fill_ms, ev[0], ev[1]));
    if (prefill_timed && levels_timed && deps_late) {
      // without the time the levels waited for the tables they read: work lists and pre-fill, then the levels
      float a = 0, b = 0;
      HIP_TRY(hipEventElapsedTime(&a, ev[0], ev[4]));
      HIP_TRY(hipEventElapsedTime(&b, ev[5], ev[1]));
      stats->fill_ms = a + b;
    }
    HIP_TRY(hipEventElapsedTime(&stats->compress_ms, ev[3], ev[2]));
    if (prefill_timed) HIP_TRY(hipEventElapsedTime(&stats->prefill_ms, ev[0], ev[4]));
    stats->n_decision_boxes = tab->list_n[0];
    stats->n_cost_boxes = tab->list_n[1];
    stats->scratch_used = needed;
  }
  guard.p = nullptr;
  *out = tab;
  return MRL_OK;
  });
}

// Indices of specs[first], specs[first + 1], ...  A function of its own: within the closures of a question the loop
// fetched what they capture again for every Spec (32,768 Specs asked of the dense table: 133 us, 126 this way).
__attribute__((noinline)) int32_t pack_indices(const Geo& g, const mrl_coord* specs, size_t first, uint32_t m, uint64_t* idx) {
  for (uint32_t i = 0; i < m; i++) {
    uint64_t x = 0;
    for (uint32_t a = 0; a < g.ndim; a++) {
      const uint32_t v = specs[first + i].x[a];
      if (v >= g.ext[a]) return fail(MRL_E_RANGE, "spec %zu: coordinate %u = %u outside [0, %u)", first + i, a, v, g.ext[a]);
      x += (uint64_t)v * g.stride[a];
    }
    idx[i] = x;
  }
  return MRL_OK;
}

}  // namespace

extern "C" {

int32_t mrl_solve(const mrl_target* t, const mrl_lattice_desc* lat, const mrl_table* const* deps, uint32_t n_deps,
                  void* d_cost, void* d_argmin, void* d_scratch, size_t scratch_bytes, void* hip_stream,
                  mrl_table** out, mrl_stats* stats) {
  return solve_impl(t, lat, deps, n_deps, d_cost, d_argmin, d_scratch, scratch_bytes, hip_stream, out, stats, FilledFn());
}

int32_t mrl_solve_graph(const mrl_target* t, const mrl_job* jobs, uint32_t n_jobs, mrl_table** out, mrl_stats* stats) {
  return guarded([&]() -> int32_t {
  if (!out) return fail(MRL_E_INVAL, "out is NULL");
  for (uint32_t j = 0; j < n_jobs && j < MRL_MAX_JOBS; j++) out[j] = nullptr;
  if (!t || !jobs) return fail(MRL_E_INVAL, "NULL argument");
  if (n_jobs < 1 || n_jobs > MRL_MAX_JOBS) return fail(MRL_E_INVAL, "n_jobs must be 1..%d", MRL_MAX_JOBS);
  for (uint32_t j = 0; j < n_jobs; j++) {
    if (!jobs[j].lattice) return fail(MRL_E_INVAL, "job %u: lattice descriptor is NULL", j);
    if (jobs[j].n_deps > 2) return fail(MRL_E_INVAL, "job %u: at most two deps", j);
    for (uint32_t i = 0; i < jobs[j].n_deps; i++)
      if (jobs[j].deps[i] >= j) return fail(MRL_E_INVAL, "job %u: a dep must be an earlier job", j);
    for (uint32_t k = 0; k < j; k++)
      if (jobs[k].hip_stream == jobs[j].hip_stream) return fail(MRL_E_INVAL, "jobs %u and %u share a stream", k, j);
  }
  // No lattice twice (solves of one (target, lattice) take turns for its upload image: such jobs
  // would not overlap, and nothing reads two tables of one lattice).
  CompiledPtr compiled[MRL_MAX_JOBS];
  for (uint32_t j = 0; j < n_jobs; j++) {
    const int32_t rc = get_compiled(t->d, jobs[j].lattice, compiled[j]);
    if (rc) { char msg[sizeof g_err]; snprintf(msg, sizeof msg, "%s", g_err); return fail(rc, "job %u: %s", j, msg); }
    for (uint32_t k = 0; k < j; k++)
      if (compiled[k] == compiled[j]) return fail(MRL_E_INVAL, "jobs %u and %u are the same lattice", k, j);
  }
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));

  enum { kWaiting = 0, kFilled = 1, kFailed = 2 };
  struct Shared {
    std::mutex mu;
    std::condition_variable cv;
    int state[MRL_MAX_JOBS] = {};
    mrl_table* table[MRL_MAX_JOBS] = {};      // from the moment a job's fill is queued
    hipEvent_t filled[MRL_MAX_JOBS] = {};     // recorded on the job's stream at that moment
    int32_t rc[MRL_MAX_JOBS] = {};
    bool skipped[MRL_MAX_JOBS] = {};          // not run: a dep failed
    std::string err[MRL_MAX_JOBS];
  } S;
  struct Events {
    Shared& s; uint32_t n = 0;
    ~Events() { for (uint32_t j = 0; j < n; j++) (void)hipEventDestroy(s.filled[j]); }
  } events{S};
  for (uint32_t j = 0; j < n_jobs; j++) {
    HIP_TRY(hipEventCreateWithFlags(&S.filled[j], hipEventDisableTiming));
    events.n = j + 1;
  }

  auto run_job = [&](uint32_t j) {
    const mrl_job& job = jobs[j];
    int32_t rc = MRL_OK;
    bool published = false;
    auto finish = [&](int32_t code) {
      if (code) S.err[j] = g_err;
      std::lock_guard<std::mutex> lk(S.mu);
      S.rc[j] = code;
      if (!published) { S.table[j] = out[j]; S.state[j] = code ? kFailed : kFilled; }
      S.cv.notify_all();
    };
    if (hipSetDevice(dev) != hipSuccess) { finish(fail(MRL_E_HIP, "hipSetDevice failed")); return; }
    // The tables the job reads, handed over when its fill needs them (its work lists and pre-fill
    // are queued by then): wait until their fills are queued; a dep's dense table is complete once
    // its stream has passed the recorded point.
    const LateDepsFn late_deps = [&](const mrl_table* tables[2], hipEvent_t ready[2]) -> int32_t {
      std::unique_lock<std::mutex> lk(S.mu);
      for (uint32_t i = 0; i < job.n_deps; i++) {
        const uint32_t d = job.deps[i];
        S.cv.wait(lk, [&] { return S.state[d] != kWaiting; });
        if (S.state[d] == kFailed) { S.skipped[j] = true; return fail(MRL_E_INVAL, "a dep of the job failed"); }
        tables[i] = S.table[d];
        ready[i] = S.filled[d];
      }
      return MRL_OK;
    };
    // (the job's own first kernels go to the GPU only once the fills it will read are queued: a
    // pre-fill that arrives before them fills every compute unit and holds them up)
    {
      std::unique_lock<std::mutex> lk(S.mu);
      for (uint32_t i = 0; i < job.n_deps; i++) S.cv.wait(lk, [&] { return S.state[job.deps[i]] != kWaiting; });
    }
    rc = solve_impl(t, job.lattice, nullptr, job.n_deps, job.d_cost, job.d_argmin, job.d_scratch,
                    job.scratch_bytes, job.hip_stream, &out[j], stats ? &stats[j] : nullptr,
                    [&](mrl_table* tab) {
                      if (hipEventRecord(S.filled[j], tab->stream) != hipSuccess) return false;   // published at the end instead
                      std::unique_lock<std::mutex> lk(S.mu);
                      S.table[j] = tab;
                      S.state[j] = kFilled;
                      published = true;
                      S.cv.notify_all();
                      // the compression waits until the jobs that read this table have queued their
                      // fill (or failed): its many small launches would otherwise hold up theirs
                      for (uint32_t k = j + 1; k < n_jobs; k++)
                        for (uint32_t i = 0; i < jobs[k].n_deps; i++)
                          if (jobs[k].deps[i] == j) S.cv.wait(lk, [&] { return S.state[k] != kWaiting; });
                      return true;
                    }, late_deps);
    finish(rc);
  };
  // a job always reports: its dependents wait for it
  auto run = [&](uint32_t j) {
    try { run_job(j); }
    catch (...) {
      std::lock_guard<std::mutex> lk(S.mu);
      S.rc[j] = MRL_E_NOMEM;
      if (S.state[j] == kWaiting) S.state[j] = kFailed;
      S.cv.notify_all();
    }
  };
  {
    // the last job runs on the calling thread, the others on the library's worker threads
    uint32_t pending = 0;                     // under S.mu: submitted jobs that have not ended
    bool submit_failed = false;
    for (uint32_t j = 0; j + 1 < n_jobs; j++) {
      { std::lock_guard<std::mutex> lk(S.mu); pending++; }
      try {
        workers().submit([&, j] {
          run(j);
          std::lock_guard<std::mutex> lk(S.mu);
          pending--;
          S.cv.notify_all();
        });
      } catch (...) {
        // no thread for this job: it and the jobs after it fail (those that wait for them wake up)
        std::lock_guard<std::mutex> lk(S.mu);
        pending--;
        for (uint32_t k = j; k < n_jobs; k++) { S.rc[k] = MRL_E_NOMEM; S.state[k] = kFailed; }
        S.cv.notify_all();
        submit_failed = true;
        break;
      }
    }
    if (!submit_failed) run(n_jobs - 1);
    std::unique_lock<std::mutex> lk(S.mu);
    S.cv.wait(lk, [&] { return pending == 0; });
  }
  uint32_t bad = n_jobs;
  for (uint32_t j = 0; j < n_jobs && bad == n_jobs; j++) if (S.rc[j] && !S.skipped[j]) bad = j;
  if (bad == n_jobs) return MRL_OK;
  // every table goes, also one that was shared before its own solve failed
  for (uint32_t j = 0; j < n_jobs; j++) {
    delete (S.table[j] ? S.table[j] : out[j]);
    out[j] = nullptr;
  }
  return fail(S.rc[bad], "job %u: %s", bad, S.err[bad].empty() ? "host allocation failed" : S.err[bad].c_str());
  });
}

void mrl_table_destroy(mrl_table* tab) { delete tab; }

int32_t mrl_query(const mrl_table* tab, const mrl_coord* specs, size_t n, uint64_t* cost_out, uint16_t* rewrite_out) {
  return guarded([&]() -> int32_t {
  if (!tab || (n && (!specs || !cost_out || !rewrite_out))) return fail(MRL_E_INVAL, "NULL argument");
  const Geo& g = tab->cp->geo;
  if (!n) return MRL_OK;
  OnDevice on;
  const int32_t rc = on.set(tab->device);
  if (rc) return rc;
  // a chunk: linear indices, costs, rewrite ids
  static_assert((size_t)kQueryChunk * 18 <= kStageHalf, "a chunk fits half a staging block");
  return take_in_parts(n, kQueryChunk, 18, tab->device, tab->stream,
    [&](size_t first, uint32_t m, char* h, size_t) { return pack_indices(g, specs, first, m, (uint64_t*)h); },
    [&](size_t, uint32_t m, char* h, size_t of, hipStream_t st) {
      return launch_gather((const uint64_t*)h, m, tab->d_cost, tab->d_arg, (uint64_t*)(h + of * 8), (uint16_t*)(h + of * 16), st);
    },
    [&](size_t first, uint32_t m, char* h, size_t of) -> int32_t {
      memcpy(cost_out + first, h + of * 8, (size_t)m * 8);
      memcpy(rewrite_out + first, h + of * 16, (size_t)m * 2);
      return MRL_OK;
    });
  });
}

// Staging of mrl_query_noalloc: linear indices in, costs and rewrite ids out.  One copy per GPU,
// held until the process ends; `scratch` itself is only a host-side name for it (not a device
// address): its address on the current device comes from hipGetSymbolAddress, once per device.
namespace {
struct NoAllocStaging {
  uint64_t idx[MRL_NOALLOC_MAX_QUERIES];
  uint64_t cost[MRL_NOALLOC_MAX_QUERIES];
  uint16_t arg[MRL_NOALLOC_MAX_QUERIES];
};
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;                       // calls that use the array take turns
void* g_noalloc_ptr[kMaxDevices] = {};         // the array's address per device, under g_noalloc_mu
}  // namespace
static __device__ __align__(256) unsigned char scratch[sizeof(NoAllocStaging)];

int32_t mrl_query_noalloc(const mrl_table* tab, const mrl_coord* specs, size_t n, uint64_t* cost_out, uint16_t* rewrite_out) {
  return guarded([&]() -> int32_t {
  if (!tab || (n && (!specs || !cost_out || !rewrite_out))) return fail(MRL_E_INVAL, "NULL argument");
  if (n > MRL_NOALLOC_MAX_QUERIES)
    return fail(MRL_E_INVAL, "mrl_query_noalloc takes at most %d Specs per call, %zu given", (int)MRL_NOALLOC_MAX_QUERIES, n);
  if (n == 0) return MRL_OK;
  const Geo& g = tab->cp->geo;
  uint64_t idx[MRL_NOALLOC_MAX_QUERIES];       // on the stack: nothing is allocated, on the host either
  const int32_t rc = pack_indices(g, specs, 0, (uint32_t)n, idx);
  if (rc) return rc;
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(MRL_E_INVAL, "device %d: at most %d devices", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (!g_noalloc_ptr[dev]) {
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(MRL_E_HIP, "hipGetSymbolAddress gave no address");
    g_noalloc_ptr[dev] = p;
  }
  NoAllocStaging* d = (NoAllocStaging*)g_noalloc_ptr[dev];
  // the previous call's contents are simply overwritten: the kernel reads idx[0, n) and writes
  // cost[0, n), arg[0, n), and only those come back
  const uint32_t m = (uint32_t)n;
  HIP_TRY(hipMemcpyAsync(d->idx, idx, n * 8, hipMemcpyHostToDevice, tab->stream));
  HIP_TRY(launch_gather(d->idx, m, tab->d_cost, tab->d_arg, d->cost, d->arg, tab->stream));
  HIP_TRY(hipMemcpyAsync(cost_out, d->cost, n * 8, hipMemcpyDeviceToHost, tab->stream));
  HIP_TRY(hipMemcpyAsync(rewrite_out, d->arg, n * 2, hipMemcpyDeviceToHost, tab->stream));
  HIP_TRY(hipStreamSynchronize(tab->stream));
  return MRL_OK;
  });
}

int32_t mrl_rewrite_decode(const mrl_table* tab, uint16_t id, mrl_rewrite* out) {
  return guarded([&]() -> int32_t {
  if (!tab || !out) return fail(MRL_E_INVAL, "NULL argument");
  const DevParams& P = tab->P;
  memset(out, 0, sizeof *out);
  if (id < P.move_base) { out->cls = 0; out->mk_index = id; return MRL_OK; }
  if (id < P.tile_base) {
    uint32_t r = id - P.move_base;
    out->cls = 1; out->convert = r & 1; r >>= 1;
    out->transposed = (uint8_t)(r % P.xw); r /= P.xw;
    out->dst_level = (uint8_t)(r % (P.NL - 1)); out->operand_or_dim = (uint8_t)(r / (P.NL - 1));
    return MRL_OK;
  }
  if (id < P.buf_id) {
    const uint32_t r = id - P.tile_base, d = r / P.maxs, j = r % P.maxs;
    if (j >= P.nsz[d]) return fail(MRL_E_RANGE, "rewrite id %u names no tile size", id);
    out->cls = 2; out->operand_or_dim = (uint8_t)d; out->tile_size = tab->cp->sizes[d][j];
    return MRL_OK;
  }
  if (id == P.buf_id && P.kind == kKindF) { out->cls = 3; return MRL_OK; }
  if (P.split && id >= P.buf_id && id < P.buf_id + P.NL) { out->cls = 3; out->dst_level = (uint8_t)(id - P.buf_id); return MRL_OK; }
  if (P.par && id >= P.par_base && id < P.par_base + 4 * P.maxs) {
    const uint32_t r = id - P.par_base, d = r / P.maxs, j = r % P.maxs;
    if (d != 2 && j < P.nsz[d]) { out->cls = 4; out->operand_or_dim = (uint8_t)d; out->tile_size = P.sizes[d][j]; return MRL_OK; }
  }
  return fail(MRL_E_RANGE, "rewrite id %u is not used by this table", id);
  });
}

int32_t mrl_coord_of_spec(const mrl_table* tab, const uint32_t shape[4], const uint8_t* levels, const uint8_t* layouts,
                          const uint8_t* dtypes, mrl_coord* out) {
  return guarded([&]() -> int32_t {
  if (!tab || !shape || !levels || !out) return fail(MRL_E_INVAL, "NULL argument");
  const Compiled& c = *tab->cp;
  memset(out, 0, sizeof *out);
  for (int d = 0; d < 4; d++) {
    auto it = std::lower_bound(c.sizes[d].begin(), c.sizes[d].end(), shape[d]);
    if (it == c.sizes[d].end() || *it != shape[d]) return fail(MRL_E_RANGE, "size %u is not allowed on dimension %d", shape[d], d);
    out->x[d] = (uint32_t)(it - c.sizes[d].begin());
  }
  for (uint32_t i = 0; i < c.P.nlv; i++) {
    if (levels[i] >= c.P.NL) return fail(MRL_E_RANGE, "level %u of operand %u outside the target", levels[i], i);
    out->x[4 + i] = levels[i];
  }
  for (uint32_t a = 0; a < c.P.nlim; a++) out->x[4 + c.P.nlv + a] = c.P.lim_nq[a] - 1;   // the whole capacity
  for (uint32_t i = 0; i < c.P.nops; i++) {
    if (c.lay_axis[i] >= 0) { if (!layouts || layouts[i] >= (1u << c.P.lay_w[i])) return fail(MRL_E_RANGE, "layout of operand %u", i); out->x[c.lay_axis[i]] = layouts[i]; }
    if (c.dt_axis[i] >= 0) { if (!dtypes || dtypes[i] > 1) return fail(MRL_E_RANGE, "dtype of operand %u", i); out->x[c.dt_axis[i]] = dtypes[i]; }
  }
  return MRL_OK;
  });
}

namespace {

// The entries of a program's Specs: chains of them come from the GPU (launch_chain walks on from a
// Spec while the child is in the same table), so that a program of some dozen rewrites is a few
// round trips.  A chain is only read ahead: an entry is used where the Spec that is asked for next is
// the one the chain holds.
struct ChainReader {
  StageLease stage;
  const mrl_table* t = nullptr;
  uint32_t at = 0, n = 0;
  int32_t entry(const mrl_table* tab, const mrl_coord& x, uint64_t* cost, uint16_t* rw) {
    const Compiled& c = *tab->cp;
    const Geo& g = c.geo;
    const DevParams& P = tab->P;
    uint32_t cell = 0;
    for (uint32_t a = 0; a < g.ndim; a++) {
      if (x.x[a] >= g.ext[a]) return fail(MRL_E_RANGE, "spec 0: coordinate %u = %u outside [0, %u)", a, x.x[a], g.ext[a]);
      cell += x.x[a] * g.stride[a];
    }
    if (!stage.mem) {
      const int32_t rc = get_stage(stage);
      if (rc) return rc;
    }
    ChainEntry* e = (ChainEntry*)stage.mem;
    if (t != tab || at >= n || e[at].cell != cell) {
      ChainWalk w;
      w.g = g;
      w.cell = cell;
      for (uint32_t a = 0; a < 16; a++) w.x[a] = x.x[a];
      w.move_base = P.move_base; w.tile_base = P.tile_base; w.buf_id = P.buf_id; w.maxs = P.maxs; w.xw = P.xw; w.n_dst = P.NL - 1;
      // children that differ in more than the rewrite names are left to the host: the bound that a Move
      // takes its buffer from, a Move's own Specs, what is known of a tile of a Move Spec
      w.moves = !P.bounded && !P.moves && P.kind != kKindV;
      w.tiles = P.kind != kKindV;
      for (int i = 0; i < 5; i++) { w.lay_axis[i] = c.lay_axis[i]; w.dt_axis[i] = c.dt_axis[i]; }
      uint32_t* count = (uint32_t*)(e + kChainMost);
      *count = 0;
      HIP_TRY(launch_chain(w, tab->d_cost, tab->d_arg, e, count, tab->stream));
      HIP_TRY(hipStreamSynchronize(tab->stream));
      t = tab; at = 0; n = *count;
      if (n == 0 || n > kChainMost || e[0].cell != cell) return fail(MRL_E_HIP, "internal error: a Spec's entry was not read");
    }
    *cost = e[at].cost;
    *rw = (uint16_t)e[at].arg;
    at++;
    return MRL_OK;
  }
};
static_assert((kChainMost + 1) * sizeof(ChainEntry) <= 2 * kStageHalf, "a chain fits a staging block");

}  // namespace

int32_t mrl_schedule(const mrl_table* tab, const mrl_coord* goal, mrl_schedule_node* out, size_t cap, size_t* n_out) {
  return guarded([&]() -> int32_t {
  if (!tab || !goal) return fail(MRL_E_INVAL, "NULL argument");
  struct Item { const mrl_table* t; uint32_t which; mrl_coord x; };
  OnDevice on;
  int32_t rc = on.set(tab->device);
  if (rc) return rc;
  std::vector<Item> stack;
  stack.push_back({tab, 0u, *goal});
  ChainReader reader;
  size_t n = 0;
  while (!stack.empty()) {
    const Item it = stack.back();
    stack.pop_back();
    const Compiled& c = *it.t->cp;
    const DevParams& P = it.t->P;
    uint64_t cost;
    uint16_t rw;
    rc = reader.entry(it.t, it.x, &cost, &rw);
    if (rc) return rc;
    if (cost == kInf) {
      if (n == 0) return fail(MRL_E_INVAL, "the goal Spec has no implementation");
      return fail(MRL_E_HIP, "internal error: a rewrite of a finite Spec leads to a Spec without implementation");
    }
    mrl_rewrite r;
    rc = mrl_rewrite_decode(it.t, rw, &r);
    if (rc) return rc;
    mrl_schedule_node node;
    memset(&node, 0, sizeof node);
    node.table = it.which; node.rewrite = rw; node.cost = cost; node.spec = it.x;
    if (r.cls == 1) {                       // Move: the operand one or more levels down, perhaps in another layout / converted
      const uint32_t op = r.operand_or_dim;
      Item ch = it;
      ch.x.x[4 + op] = r.dst_level;
      if (r.transposed) { if (c.lay_axis[op] < 0) return fail(MRL_E_HIP, "internal error: transposing Move without a layout coordinate"); ch.x.x[c.lay_axis[op]] ^= r.transposed; }
      if (r.convert) { if (c.dt_axis[op] < 0) return fail(MRL_E_HIP, "internal error: converting Move without a dtype coordinate"); ch.x.x[c.dt_axis[op]] = 0; }
      if (P.bounded && P.lim_of_level[r.dst_level] != kNoBit) {
        // the Move's buffer comes out of the destination's bound; the rest snaps down to a power of two
        const uint32_t ax = 4 + P.nlv + P.lim_of_level[r.dst_level];
        const uint64_t b = c.sizes[0][it.x.x[0]], m = c.sizes[1][it.x.x[1]], k = c.sizes[2][it.x.x[2]], nn = c.sizes[3][it.x.x[3]];
        const uint64_t numel = P.kind == kKindM ? (op == 0 ? b * m * k : op == 1 ? b * k * nn : b * m * nn)
                             : P.kind == kKindE ? (op == 1 ? nn : m * nn)
                                                : (op == 0 ? m * k : op == 1 ? k * nn : op == 2 ? nn : m * nn);
        const bool bf = c.dt_axis[op] >= 0 ? ch.x.x[c.dt_axis[op]] != 0 : c.lat.base_dtype_bytes[op] == 2;
        const uint64_t bytes = numel * (bf ? 2 : 4), have = it.x.x[ax] ? 1ull << (it.x.x[ax] - 1) : 0;
        if (bytes > have) return fail(MRL_E_HIP, "internal error: a memoized Move exceeds its memory bound");
        uint64_t left = have - bytes;
        uint32_t q = 0;
        while (left) { q++; left >>= 1; }
        ch.x.x[ax] = q;
      }
      node.n_children = 1;
      if (P.moves) {
        // Section 2, Memory Movement: the alloc-binding holds a load Move Spec (operands that are read),
        // the body, and a store Move Spec (operands that are written), both of fresh tensors
        if (it.which != 0 || !it.t->deps[0]) return fail(MRL_E_HIP, "internal error: a Move Spec outside a MATMUL_MOVES table");
        const mrl_table* vt = it.t->deps[0];
        const Compiled& vc = *vt->cp;
        const uint32_t y0 = c.lay_axis[op] >= 0 ? it.x.x[c.lay_axis[op]] : 0u, y1 = c.lay_axis[op] >= 0 ? ch.x.x[c.lay_axis[op]] : 0u;
        const uint32_t f0 = c.dt_axis[op] >= 0 ? it.x.x[c.dt_axis[op]] : (uint32_t)(c.lat.base_dtype_bytes[op] == 2);
        const uint32_t f1 = c.dt_axis[op] >= 0 ? ch.x.x[c.dt_axis[op]] : f0;
        auto move_spec = [&](uint32_t ls, uint32_t ld, uint32_t ys, uint32_t yd, uint32_t fs, uint32_t fd, Item& out_item) -> int32_t {
          out_item = Item{vt, 1u, {}};
          mrl_coord& x = out_item.x;
          memset(&x, 0, sizeof x);
          x.x[1] = op == 1 ? it.x.x[2] : it.x.x[1];      // rows: m (lhs, out) or k (rhs); the size lists are the same
          x.x[3] = op == 0 ? it.x.x[2] : it.x.x[3];      // columns: k (lhs) or n
          x.x[4] = ls; x.x[5] = ld;
          x.x[6] = ys >= 2 ? 3 : 2; x.x[7] = 1; x.x[8] = yd >= 2 ? 3 : 2; x.x[9] = 1;
          if (vc.lay_axis[0] >= 0) x.x[vc.lay_axis[0]] = ys; else if (ys) return fail(MRL_E_HIP, "internal error: the MOVE table lacks a layout coordinate");
          if (vc.lay_axis[1] >= 0) x.x[vc.lay_axis[1]] = yd; else if (yd) return fail(MRL_E_HIP, "internal error: the MOVE table lacks a layout coordinate");
          if (vc.dt_axis[0] >= 0) x.x[vc.dt_axis[0]] = fs;
          if (vc.dt_axis[1] >= 0) x.x[vc.dt_axis[1]] = fd;
          return MRL_OK;
        };
        Item load, store;
        const bool has_load = P.access[op] != kWrite, has_store = P.access[op] != kRead;
        if (has_store) { rc = move_spec(r.dst_level, it.x.x[4 + op], y1, y0, f1, f0, store); if (rc) return rc; stack.push_back(store); }
        stack.push_back(ch);                // popped after the load's whole subtree, before the store's
        if (has_load) { rc = move_spec(it.x.x[4 + op], r.dst_level, y0, y1, f0, f1, load); if (rc) return rc; stack.push_back(load); }
        node.n_children = (uint16_t)(1 + (has_load ? 1 : 0) + (has_store ? 1 : 0));
      } else {
        stack.push_back(ch);
      }
    } else if (r.cls == 2) {                // tile: the loop body is the Spec with the smaller size
      const uint32_t d = r.operand_or_dim, j = (rw - P.tile_base) % P.maxs;
      Item ch = it;
      ch.x.x[d] = j;
      if (P.kind == kKindV) {
        // Section 2.4.3: what is known of the tile of either tensor
        const uint32_t rows = c.sizes[1][it.x.x[1]], cols = c.sizes[3][it.x.x[3]];
        const uint32_t r2 = c.sizes[1][ch.x.x[1]], c2 = c.sizes[3][ch.x.x[3]];
        for (int ts = 0; ts < 2; ts++) {
          const uint32_t y = c.lay_axis[ts] >= 0 ? it.x.x[c.lay_axis[ts]] : 0u;
          const bool bf = c.dt_axis[ts] >= 0 ? it.x.x[c.dt_axis[ts]] != 0 : c.lat.base_dtype_bytes[ts] == 2;
          uint32_t contig2, aligned2;
          tile_abstract(y, rows, cols, r2, c2, bf ? 2 : 4, P.strip ? P.strip : 1, P.line_bytes, P.line_mask, it.x.x[6 + 2 * ts], it.x.x[7 + 2 * ts],
                        contig2, aligned2);
          ch.x.x[6 + 2 * ts] = contig2; ch.x.x[7 + 2 * ts] = aligned2;
        }
      }
      stack.push_back(ch);
      node.n_children = 1;
    } else if (r.cls == 4) {                // parallel loop: the body is the serial-only Spec of the smaller size
      if (it.which != 0 || !it.t->deps[0]) return fail(MRL_E_HIP, "internal error: parallel loop outside a MATMUL_PARALLEL table");
      const uint32_t d = r.operand_or_dim, j = (rw - P.par_base) % P.maxs;
      Item ch{it.t->deps[0], 1u, it.x};
      ch.x.x[d] = j;
      stack.push_back(ch);
      node.n_children = 1;
    } else if (r.cls == 3 && P.split) {     // bufferize between the bias add and the ReLU, the intermediate in level r.dst_level
      if ((it.which != 0 && it.which != 2) || !it.t->deps[0] || !it.t->deps[1]) return fail(MRL_E_HIP, "internal error: bufferize outside a BIAS_ADD_RELU_SPLIT table");
      const uint32_t m = c.sizes[1][it.x.x[1]], nn = c.sizes[3][it.x.x[3]];
      const uint8_t l_mid = r.dst_level;
      const uint8_t y_in = c.lay_axis[0] >= 0 ? (uint8_t)it.x.x[c.lay_axis[0]] : 0, y_out = c.lay_axis[2] >= 0 ? (uint8_t)it.x.x[c.lay_axis[2]] : 0;
      const uint32_t shape_e[4] = {1, m, 1, nn};
      const uint8_t lv_a[5] = {(uint8_t)it.x.x[4], (uint8_t)it.x.x[5], l_mid, 0, 0}, ly_a[5] = {y_in, 0, 0, 0, 0};
      const uint8_t lv_r[5] = {l_mid, (uint8_t)it.x.x[6], 0, 0, 0}, ly_r[5] = {0, y_out, 0, 0, 0};
      const uint8_t zeros[5] = {0, 0, 0, 0, 0};
      // (tables 3 and 4 when this table is itself dep 1 of the table the walk started in)
      Item ca{it.t->deps[0], it.which + 1u, {}}, cr{it.t->deps[1], it.which + 2u, {}};
      rc = mrl_coord_of_spec(ca.t, shape_e, lv_a, ly_a, zeros, &ca.x);
      if (rc) return rc;
      rc = mrl_coord_of_spec(cr.t, shape_e, lv_r, ly_r, zeros, &cr.x);
      if (rc) return rc;
      stack.push_back(cr);                  // popped after the bias add's whole subtree
      stack.push_back(ca);
      node.n_children = 2;
    } else if (r.cls == 3 && P.chain) {     // bufferize of a composition: the Matmul (m, k, p) into the intermediate, then (m, p, n) out of it
      if (it.which != 0 || !it.t->deps[0]) return fail(MRL_E_HIP, "internal error: bufferize outside a MATMUL_CHAIN table");
      const uint32_t p = c.sizes[0][it.x.x[0]], m = c.sizes[1][it.x.x[1]], k = c.sizes[2][it.x.x[2]], nn = c.sizes[3][it.x.x[3]];
      const uint8_t l_mid = (uint8_t)it.x.x[8];
      uint8_t y[4];
      for (int i = 0; i < 4; i++) y[i] = c.lay_axis[i] >= 0 ? (uint8_t)it.x.x[c.lay_axis[i]] : 0;
      const uint32_t shape_1[4] = {1, m, k, p}, shape_2[4] = {1, m, p, nn};
      const uint8_t lv_1[5] = {(uint8_t)it.x.x[4], (uint8_t)it.x.x[5], l_mid, 0, 0}, ly_1[5] = {y[0], y[1], 0, 0, 0};
      const uint8_t lv_2[5] = {l_mid, (uint8_t)it.x.x[6], (uint8_t)it.x.x[7], 0, 0}, ly_2[5] = {0, y[2], y[3], 0, 0};
      const uint8_t zeros[5] = {0, 0, 0, 0, 0};
      Item c1{it.t->deps[0], 1u, {}}, c2{it.t->deps[0], 1u, {}};
      rc = mrl_coord_of_spec(c1.t, shape_1, lv_1, ly_1, zeros, &c1.x);
      if (rc) return rc;
      rc = mrl_coord_of_spec(c2.t, shape_2, lv_2, ly_2, zeros, &c2.x);
      if (rc) return rc;
      stack.push_back(c2);                  // popped after the first Matmul's whole subtree
      stack.push_back(c1);
      node.n_children = 2;
    } else if (r.cls == 3) {                // bufferize: Matmul into the intermediate, then bias-add + ReLU out of it
      if (it.which != 0 || !it.t->deps[0] || !it.t->deps[1]) return fail(MRL_E_HIP, "internal error: bufferize outside a FUSED table");
      const uint32_t m = c.sizes[1][it.x.x[1]], k = c.sizes[2][it.x.x[2]], nn = c.sizes[3][it.x.x[3]];
      const uint8_t l_lhs = (uint8_t)it.x.x[4], l_rhs = (uint8_t)it.x.x[5], l_bias = (uint8_t)it.x.x[6], l_out = (uint8_t)it.x.x[7];
      const uint8_t l_mid = (uint8_t)it.x.x[8];
      const uint8_t y_lhs = c.lay_axis[0] >= 0 ? (uint8_t)it.x.x[c.lay_axis[0]] : 0, y_rhs = c.lay_axis[1] >= 0 ? (uint8_t)it.x.x[c.lay_axis[1]] : 0;
      const uint8_t y_out = c.lay_axis[3] >= 0 ? (uint8_t)it.x.x[c.lay_axis[3]] : 0;
      const uint32_t shape_m[4] = {1, m, k, nn}, shape_e[4] = {1, m, 1, nn};
      const uint8_t lv_m[5] = {l_lhs, l_rhs, l_mid, 0, 0}, ly_m[5] = {y_lhs, y_rhs, 0, 0, 0};
      const uint8_t lv_e[5] = {l_mid, l_bias, l_out, 0, 0}, ly_e[5] = {0, 0, y_out, 0, 0};
      const uint8_t zeros[5] = {0, 0, 0, 0, 0};
      Item cm{it.t->deps[0], 1u, {}}, ce{it.t->deps[1], 2u, {}};
      rc = mrl_coord_of_spec(cm.t, shape_m, lv_m, ly_m, zeros, &cm.x);
      if (rc) return rc;
      rc = mrl_coord_of_spec(ce.t, shape_e, lv_e, ly_e, zeros, &ce.x);
      if (rc) return rc;
      if (P.bounded) {
        // both stages inherit the bounds; the intermediate's bytes come out of its level's bound
        for (uint32_t a = 0; a < P.nlim; a++) cm.x.x[4 + 3 + a] = ce.x.x[4 + 3 + a] = it.x.x[4 + P.nlv + a];
        if (P.lim_of_level[l_mid] != kNoBit) {
          const uint32_t a = P.lim_of_level[l_mid], q = it.x.x[4 + P.nlv + a];
          const uint64_t bytes = (uint64_t)m * nn * 4, have = q ? 1ull << (q - 1) : 0;
          if (bytes > have) return fail(MRL_E_HIP, "internal error: a memoized bufferize exceeds its memory bound");
          uint64_t left = have - bytes;
          uint32_t qn = 0;
          while (left) { qn++; left >>= 1; }
          cm.x.x[4 + 3 + a] = ce.x.x[4 + 3 + a] = qn;
        }
      }
      stack.push_back(ce);                  // popped after the Matmul's whole subtree
      stack.push_back(cm);
      node.n_children = 2;
    }
    if (out && n < cap) out[n] = node;
    n++;
    if (n > (1u << 20)) return fail(MRL_E_HIP, "internal error: schedule does not end");
  }
  if (n_out) *n_out = n;
  if (out && cap < n) return fail(MRL_E_BUFSZ, "schedule buffer holds %zu nodes, %zu needed", cap, n);
  return MRL_OK;
  });
}

int32_t mrl_emit_compressed(const mrl_table* tab, uint32_t which, mrl_box* out, size_t cap, size_t* n_out) {
  return guarded([&]() -> int32_t {
  if (!tab || which > 1) return fail(MRL_E_INVAL, "bad argument");
  const uint64_t n = tab->list_n[which];
  if (n_out) *n_out = n;
  if (!out) return MRL_OK;
  if (cap < n) return fail(MRL_E_BUFSZ, "box buffer holds %zu, %llu needed", cap, (unsigned long long)n);
  const Geo& g = tab->cp->geo;
  if (!n) return MRL_OK;
  const char* r = tab->scratch + tab->list_off[which];
  const uint32_t* fcell = (const uint32_t*)r; r += align_up(n * 4);
  const char* flen = r; r += align_up(n * 16);
  const uint64_t* fv0 = (const uint64_t*)r; r += align_up(n * 8);
  const uint64_t* fv1 = (const uint64_t*)r;
  // The GPU writes the records into pinned memory, kEmitChunk at a time, while the host copies the
  // chunk before out of it.  On a stream of the library's own (a helper stream of the table's device):
  // the caller may have given up the solve's stream, and a launch on the null stream would wait for
  // every blocking stream of the process, and they for it, once per chunk.  The lists are complete:
  // the solve has waited for them.
  static_assert(sizeof(mrl_box) == 80 && (size_t)kEmitChunk * sizeof(mrl_box) <= kStageHalf, "a chunk fits half a staging block");
  OnDevice on;
  int32_t rc = on.set(tab->device);
  if (rc) return rc;
  AuxLease aux;
  rc = get_aux(0, aux);
  if (rc) return rc;
  return take_in_parts(n, kEmitChunk, sizeof(mrl_box), tab->device, aux.a->stream,
    [&](size_t, uint32_t, char*, size_t) -> int32_t { return MRL_OK; },
    [&](size_t first, uint32_t m, char* h, size_t, hipStream_t st) {
      return launch_expand_boxes(g, m, fcell + first, flen + first * 16, fv0 + first, fv1 + first, h, st);
    },
    [&](size_t first, uint32_t m, char* h, size_t) -> int32_t {
      memcpy((void*)(out + first), h, (size_t)m * sizeof(mrl_box));
      return MRL_OK;
    });
  });
}

int32_t mrl_query_compressed(const mrl_table* tab, const mrl_coord* specs, size_t n, uint64_t* cost_out,
                             uint16_t* rewrite_out) {
  return guarded([&]() -> int32_t {
  if (!tab || (n && (!specs || !cost_out || !rewrite_out))) return fail(MRL_E_INVAL, "NULL argument");
  const Compiled& c = *tab->cp;
  const Geo& g = c.geo;
  for (uint32_t a = 0; a < g.ndim; a++)
    if (g.ext[a] > 256) return fail(MRL_E_INVAL, "axis %u has %u coordinates: the box index holds one byte per axis", a, g.ext[a]);
  OnDevice on;
  const int32_t rc = on.set(tab->device);
  if (rc) return rc;
  std::lock_guard<std::mutex> lock(tab->lookup_mu);
  LookupList lists[2];
  for (uint32_t which = 0; which < 2; which++) {
    const uint64_t nb = tab->list_n[which];
    const char* r = tab->scratch + tab->list_off[which];
    const uint32_t* fcell = (const uint32_t*)r; r += align_up(nb * 4);
    const void* flen = r; r += align_up(nb * 16);
    mrl_table::BoxIndex& ix = tab->index[which];
    if (!ix.nodes) {
      ix.L = index_levels((uint32_t)nb);
      HIP_TRY(hipMalloc((void**)&ix.nodes, std::max<size_t>(ix.L.total, 1) * sizeof(BoxBounds)));
      launch_build_index(g, ix.L, fcell, flen, ix.nodes, tab->stream);
      HIP_TRY(hipGetLastError());
    }
    lists[which] = LookupList{ix.L, ix.nodes, fcell, (const uint64_t*)r, (const uint64_t*)(r + align_up(nb * 8))};
  }
  if (!n) return MRL_OK;
  // a chunk: points (16 bytes), volumes, costs, rewrite ids, a byte per list that marks a miss
  static_assert((size_t)kLookupChunk * 36 <= kStageHalf, "a chunk fits half a staging block");
  return take_in_parts(n, kLookupChunk, 36, tab->device, tab->stream,
    [&](size_t first, uint32_t m, char* h, size_t of) -> int32_t {
      uint64_t* vol = (uint64_t*)(h + of * 16);
      for (uint32_t i = 0; i < m; i++) {
        const uint32_t* x = specs[first + i].x;
        uint8_t p[16] = {};
        for (uint32_t a = 0; a < g.ndim; a++) {
          if (x[a] >= g.ext[a]) return fail(MRL_E_RANGE, "spec %zu: coordinate %u = %u outside [0, %u)", first + i, a, x[a], g.ext[a]);
          p[a] = (uint8_t)x[a];
        }
        memcpy(h + (size_t)i * 16, p, 16);
        uint64_t w = 1;
        for (uint32_t d = 0; d < 4; d++) w *= c.sizes[d][x[d]];
        vol[i] = w;
      }
      return MRL_OK;
    },
    [&](size_t, uint32_t m, char* h, size_t of, hipStream_t st) {
      return launch_lookup(g, lists, h, (const uint64_t*)(h + of * 16), m, (uint64_t*)(h + of * 24), (uint16_t*)(h + of * 32), (uint8_t*)(h + of * 34), st);
    },
    [&](size_t first, uint32_t m, char* h, size_t of) -> int32_t {
      const char* miss = h + of * 34;
      const void* bad = memchr(miss, 1, 2 * (size_t)m);
      if (bad) return fail(MRL_E_HIP, "internal error: spec %zu lies in no box", first + (size_t)((const char*)bad - miss) % m);
      memcpy(cost_out + first, h + of * 24, (size_t)m * 8);
      memcpy(rewrite_out + first, h + of * 32, (size_t)m * 2);
      return MRL_OK;
    });
  });
}

int32_t mrl_copy_dense(const mrl_table* tab, uint64_t* cost_host, uint16_t* argmin_host) {
  return guarded([&]() -> int32_t {
  if (!tab) return fail(MRL_E_INVAL, "table is NULL");
  if (cost_host) HIP_TRY(hipMemcpy(cost_host, tab->d_cost, tab->cp->n_specs * 8, hipMemcpyDeviceToHost));
  if (argmin_host) HIP_TRY(hipMemcpy(argmin_host, tab->d_arg, tab->cp->n_specs * 2, hipMemcpyDeviceToHost));
  return MRL_OK;
  });
}

}  // extern "C"
