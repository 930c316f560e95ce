// The box merge of compress.hip for tables whose shapes are whole mask words, word by word.
//
// The same merge in the same order (along n, k, m, b, then the axes inside a shape), but no box exists before the
// end.  What the merge decides is kept as bits of 64 consecutive cells (a word: a shape has G / 64 of them, all
// axes inside a shape are bit fields of a cell's place in it):
//   H     the cell starts a run along n                     (the heads of boxes after the first pass)
//   Fk    such a head was folded into the one before it along k; Fm, Fb the same for m and b
//   T     heads left after the four size axes = H & ~Fk & ~Fm & ~Fb
// Two heads are linked when their values agree and their extents on all axes already merged agree.  Extents are
// never compared as numbers: two chains of links are equally long if they end at the same step, which is one word
// operation per step when a chain is walked from its far end.
//
// Most words of a table hold no cell that fits its levels (94 % in the largest pipeline).  Rows (the words of one k
// for all n: same b, m and place in the shape) are kept up to one past the last with a fitting cell; in a row
// beyond, every cell is (INF, NONE) and folded into the row before.  All arrays are indexed by the kept rows, their
// number stays on the GPU: nothing is read back before the merge has ended (unless the scratch may be short: row_total_kernel).
// (n, k, m, b here and below: RowGeo's axes, turned where there is one size along n.)
//
//   row_count_kernel   rows kept per plane (b, m, place), then a prefix sum
//   row_info_kernel    what a wave needs of its row
//   row_heads_kernel   a wave per row: H of both lists
//   row_agree_kernel   a wave per row: heads that agree, in value and run length, with the one before on k, m, b.  Along k
//                      that settles it: Fk
//   row_fold_*_kernel  Fm; Fb: chains along k (and m) compared, by a lane each, by a wave each where they are longer than 64
//   row_left_kernel    T, and N: its heads with an extent above 1 on some size axis (few, in the cost list); prefix sums over both
//   row_extent_kernel  the four extents of the heads in N
//   row_inner_kernel   a wave per row: heads left that agree, in value and size extents, with the one a step further on
//                      an axis inside the shape, for all those axes at once.  (No pass changes that: a head that is linked
//                      to has extent 1 on the pass's axis.)
//   shape_merge_kernel the passes over the axes inside a shape, word operations only; the heads left and their extents on those axes
//   (prefix sum over the shapes' numbers of boxes)
//   row_emit_kernel    the two final lists
// Bound by instruction issue (the kernels that compare values: 60 to 80 vector instructions a word and as many scalar
// ones; emit: the reduction of the costs) and by the latency of a few dependent reads (the others).  Config 5's fused table
// (449.5 M cells, 11.3 M that fit, in 0.42 M of 7.02 M words; 44,038 rows of 38 words kept, 1.67 M words; two lists at once), us:
// heads 80, agree 159, fold 59, left 36, extent 78, inner 253, merge 161, emit 109.
#include <hip/hip_runtime.h>
#include "compress.h"
#include "dev_params.h"

namespace mrl {

typedef unsigned long long u64;

__device__ __forceinline__ u64 lane64(u64 v, uint32_t lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), (int)lane);
  return (u64)hi << 32 | lo;
}
__device__ int write_lane(int x, int lane, int v) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ void put_lane64(u64& v, u64 x, uint32_t lane) {
  const uint32_t lo = (uint32_t)write_lane((int)(uint32_t)x, (int)lane, (int)(uint32_t)v);
  const uint32_t hi = (uint32_t)write_lane((int)(uint32_t)(x >> 32), (int)lane, (int)(uint32_t)(v >> 32));
  v = (u64)hi << 32 | lo;
}
__device__ __forceinline__ bool in_mask(u64 m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ uint32_t below(u64 m) { return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)); }

// Workgroups go to the eight dies in turn.  Work that is heavy for some sizes or levels would go to the same die
// wherever these alternate with a period of two, four or eight workgroups: aligned runs of eight are rotated, each by
// another amount.
__device__ __forceinline__ uint32_t spread_block() {
  const uint32_t i = blockIdx.x;
  return (i | 7u) < gridDim.x ? (i & ~7u) | ((i + ((i >> 3) * 0x9E3779B1u >> 29)) & 7u) : i;
}

// ---------------------------------------------------------------- where things lie
// Word arrays of the kept rows, n_rows * en words each (T, N and their ranks: both lists' one after the other), the size
// extents of N's heads, the extents inside the shape of the heads left at the end (at the ranks of T's), and `agree`.  That is
// done with when the final lists are written, which take its place: without that a caller's scratch could hold the words
// and not the lists, and everything would be done twice, here and box by box.
struct RowWords {
  u64 *H[2], *Fk[2], *Fm[2], *Fb[2], *T, *N;
  uint2* rank;               // heads of N, of T before a word's
  uint32_t* ext;
  uint16_t* inner;
  u64* agree;                // per axis inside the shape (levels, then fields by their bit): T's heads that agree with the next one
};

__host__ __device__ __forceinline__ uint64_t up256(uint64_t x) { return (x + 255) & ~255ull; }

// (16 bytes, as wide as anything is read, and not 256: a table of one word would take 3.5 KB for its arrays of 8 bytes, more
// than the scratch that suffices for its boxes one by one leaves over, and would be merged both ways)
__host__ __device__ __forceinline__ uint64_t up16(uint64_t x) { return (x + 15) & ~15ull; }

__host__ __device__ __forceinline__ uint64_t row_base_bytes(const RowGeo& g, uint64_t n_rows) {
  const uint64_t sets = 2 + (g.em > 1 ? 1 : 0) + (g.eb > 1 ? 1 : 0);
  return 2 * sets * up16(n_rows * g.en * 8) + 3 * 2 * n_rows * g.en * 8;
}
__host__ __device__ __forceinline__ uint64_t row_agree_bytes(const RowGeo& g, uint64_t n_rows) { return g.n_inner * 2 * n_rows * g.en * 8; }
__host__ __device__ __forceinline__ uint64_t row_list_bytes(uint64_t n) { return up256(n * 4) + up256(n * 16) + 2 * up256(n * 8); }
// where `agree` and then the lists lie
__host__ __device__ __forceinline__ uint64_t row_lists_at(const RowGeo& g, const uint32_t* tot) {
  return up256(row_base_bytes(g, tot[kRowsTotal]) + up16((uint64_t)tot[kLongTotal] * 4) + up16((uint64_t)tot[kHeadsTotal] * 2));
}
__host__ __device__ __forceinline__ bool words_fit(const RowGeo& g, uint64_t n_rows, uint64_t room) {
  return row_base_bytes(g, n_rows) + row_agree_bytes(g, n_rows) <= room;
}

bool row_words_fit(const RowGeo& g, uint64_t n_rows, uint64_t room) { return words_fit(g, n_rows, room); }

bool rows_always_fit(const RowGeo& g, uint64_t room) {
  // every cell a head with an extent, and a box, in both lists
  const uint64_t rows = (uint64_t)g.n_planes * g.ek, cells = rows * g.en * 64;
  const uint64_t heads_end = up256(row_base_bytes(g, rows) + up16(2 * cells * 4) + up16(2 * cells * 2));
  const uint64_t agree = row_agree_bytes(g, rows), lists = 2 * row_list_bytes(cells);
  return heads_end + (agree > lists ? agree : lists) <= room;
}

bool rows_fit(const RowGeo& g, const uint32_t* tot, uint64_t room, uint64_t list_at[2], uint64_t* end) {
  // (a kernel that found no room left the totals behind it unset: in this order)
  if (!words_fit(g, tot[kRowsTotal], room)) return false;
  list_at[0] = row_lists_at(g, tot);
  const uint64_t words_end = list_at[0] + row_agree_bytes(g, tot[kRowsTotal]);
  if (words_end > room) return false;
  list_at[1] = list_at[0] + row_list_bytes(tot[kBoxesFirst]);
  const uint64_t lists_end = list_at[1] + row_list_bytes(tot[kBoxesTotal] - tot[kBoxesFirst]);
  *end = words_end > lists_end ? words_end : lists_end;
  return *end <= room;
}

// false: the rows (or, with heads, what is kept per head) do not fit the scratch; every kernel then does nothing and the
// host finds out by the same sums.
__device__ __forceinline__ bool row_words(const RowGeo& g, const RowBufs& B, RowWords& W, bool heads = false) {
  const uint64_t n_rows = B.tot[kRowsTotal], one = up16(n_rows * g.en * 8), both = 2 * n_rows * g.en * 8;
  char* p = B.dyn;
  auto take = [&](uint64_t bytes) { char* at = p; p += bytes; return at; };
  W.H[0] = (u64*)take(one); W.H[1] = (u64*)take(one);
  W.Fk[0] = (u64*)take(one); W.Fk[1] = (u64*)take(one);
  const uint64_t for_m = g.em > 1 ? one : 0, for_b = g.eb > 1 ? one : 0;        // (not used where there is no such axis)
  W.Fm[0] = (u64*)take(for_m); W.Fm[1] = (u64*)take(for_m);
  W.Fb[0] = (u64*)take(for_b); W.Fb[1] = (u64*)take(for_b);
  W.T = (u64*)take(both);
  W.N = (u64*)take(both);
  W.rank = (uint2*)take(both);
  W.ext = (uint32_t*)p; W.inner = nullptr; W.agree = nullptr;
  if (!words_fit(g, n_rows, B.room)) return false;
  if (!heads) return true;
  W.inner = (uint16_t*)(p + up16((uint64_t)B.tot[kLongTotal] * 4));
  const uint64_t lists = row_lists_at(g, B.tot);
  W.agree = (u64*)(B.dyn + lists);
  return lists + row_agree_bytes(g, n_rows) <= B.room;
}

// Sizes along axis d of b, m, k, n.
__device__ __forceinline__ const uint32_t* axis_sizes(const RowGeo& g, const uint32_t* __restrict__ sizes, uint32_t d) { return sizes + g.axis[d] * kMaxSizes; }

// Words of a row that is not kept: every cell (INF, NONE), one run along n, folded into the row before it on k.
__device__ __forceinline__ u64 gone_word(uint32_t n) { return n == 0 ? ~0ull : 0ull; }

// ---------------------------------------------------------------- rows
// Sizes ascend, and what fits a level at some size fits it at every smaller one (a layout that only some sizes have
// shares its word with the row-major one, which all have): a row has a fitting cell if its first step has one.
__device__ __forceinline__ uint32_t rows_kept(const RowGeo& g, const u64* __restrict__ fit, uint32_t p) {
  const uint32_t w = p & (g.nw - 1u), bm = p >> g.lg_nw;
  const u64* f = fit + (((size_t)bm * g.ek * g.en) << g.lg_nw) + w;
  const size_t step = (size_t)g.en << g.lg_nw;
  uint32_t last = 0;
#pragma unroll 8
  for (uint32_t k = 0; k < g.ek; k++) last = f[k * step] ? k + 1u : last;
  return last + 1u < g.ek ? last + 1u : g.ek;
}

__global__ __launch_bounds__(256) void row_count_kernel(const RowGeo g, const u64* __restrict__ fit, uint32_t* __restrict__ rows) {
  const uint32_t p = blockIdx.x * 256u + threadIdx.x;
  if (p < g.n_planes) rows[p] = rows_kept(g, fit, p);
}

// Only their number, added to *total: all that is known before the fill, whose lists lie where the rows' will.
__global__ __launch_bounds__(256) void row_total_kernel(const RowGeo g, const u64* __restrict__ fit, uint32_t* __restrict__ total) {
  const uint32_t p = blockIdx.x * 256u + threadIdx.x;
  uint32_t n = p < g.n_planes ? rows_kept(g, fit, p) : 0u;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) n += __shfl_down(n, d, 64);
  if ((threadIdx.x & 63u) == 0) atomicAdd(total, n);
}

// Cells whose normalised costs agree: c1 / s1 == c2 / s2, exactly.  i1, i2: the cells that are INF (finite costs stay
// below 2^62).  The 24-bit products settle most words; wide products take quarter-rate instructions, half as many where
// all costs are below 2^32.
__device__ __forceinline__ u64 equal_costs(uint64_t c1, uint32_t s1, u64 i1, uint64_t c2, uint32_t s2, u64 i2) {
  u64 eq = __ballot(((__umul24((uint32_t)c1, s2) ^ __umul24((uint32_t)c2, s1)) & 0xFFFFFFu) == 0) & ~(i1 | i2);
  if (eq) {
    const uint32_t h1 = (uint32_t)(c1 >> 32), h2 = (uint32_t)(c2 >> 32);
    const uint64_t l1 = (uint64_t)(uint32_t)c1 * s2, l2 = (uint64_t)(uint32_t)c2 * s1;
    if (__ballot((h1 | h2) != 0) & eq) {
      const uint64_t w1 = (uint64_t)h1 * s2 + (l1 >> 32), w2 = (uint64_t)h2 * s1 + (l2 >> 32);
      eq &= __ballot((uint32_t)l1 == (uint32_t)l2 && w1 == w2);
    } else {
      eq &= __ballot(l1 == l2);
    }
  }
  return eq | (i1 & i2);
}
__device__ __forceinline__ u64 infinite(uint64_t c) { return __ballot((uint32_t)(c >> 32) == ~0u); }

// What a wave needs of its row, worked out once: the rows it is compared with are several dependent reads away.
constexpr uint32_t kNoRow = 0xFFFFFFFFu;
struct alignas(64) RowInfo {
  uint32_t plane, k, kept;                         // kept: rows of the plane
  uint32_t m_before, m_after, b_before, b_after;   // the row one step further on an axis, kNoRow if it is not kept
  uint32_t next[kRowLevels];                       // the row of the next word on a level axis that leaves the word
  uint32_t shape0, w, b_m;                         // shape of step 0, place, b << 16 | m
  uint32_t pad;
};
static_assert(sizeof(RowInfo) == 64, "kRowInfoBytes");

__global__ __launch_bounds__(256) void row_info_kernel(const RowGeo g, const RowBufs B) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  RowInfo r;
  r.plane = i / g.ek;
  r.k = i - r.plane * g.ek;
  if (r.plane >= g.n_planes) return;
  r.kept = B.rows[r.plane];
  if (r.k >= r.kept) return;
  const uint32_t row = B.first[r.plane] + r.k;
  r.w = r.plane & (g.nw - 1u);
  const uint32_t bm = r.plane >> g.lg_nw, b = bm / g.em, m = bm - b * g.em;
  r.b_m = b << 16 | m;
  r.shape0 = (bm * g.ek + r.k) * g.en;
  auto row_of = [&](bool there, uint32_t p) { return there && r.k < B.rows[p] ? B.first[p] + r.k : kNoRow; };
  r.m_before = row_of(m > 0, r.plane - g.nw);
  r.m_after = row_of(m + 1u < g.em, r.plane + g.nw);
  r.b_before = row_of(b > 0, r.plane - g.em * g.nw);
  r.b_after = row_of(b + 1u < g.eb, r.plane + g.em * g.nw);
  for (uint32_t q = 0; q < kRowLevels; q++) {
    const uint32_t sh = g.lv + 2u * q;
    bool there = q < g.n_levels && sh >= 5u;
    if (there) there = sh == 5u ? !(r.w & 1u) : (r.w >> (sh - 6u) & 3u) < 3u;
    r.next[q] = row_of(there, r.plane + (sh >= 6u && there ? 1u << (sh - 6u) : 1u));
  }
  r.pad = 0;
  ((RowInfo*)B.info)[row] = r;
}

// The kept rows in turn, a wave each.
struct WaveRow : RowInfo {
  uint32_t row, b, m;
  __device__ __forceinline__ WaveRow(const RowBufs& B, uint32_t i) : RowInfo(((const RowInfo*)B.info)[i]), row(i) { b = b_m >> 16; m = b_m & 0xFFFFu; }
};
__device__ __forceinline__ uint32_t first_row() { return blockIdx.x * 4u + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }
constexpr uint32_t kRowGroups = 4096;     // workgroups that share the rows out
// Where there are few rows, several waves share one (its steps, its boxes), two steps a wave: every wave repeats
// what is done for the whole row.  The merge, us: with a wave a row, all sizes to 32 (at most 1,024 rows of 32 steps) 207, this 162;
// sizes 1, 2, 4, 8 with three layouts (config 5) 95, this 100, and with eight waves to a row of four steps 141.  Half the
// thresholds and three steps a wave: 16.8 M cells that all fit 521, this 509, small tables up to 8 % either way.
__device__ __forceinline__ uint32_t row_parts(const RowGeo& g, uint32_t n_rows) {
  const uint32_t most = n_rows <= 2048u ? 8u : n_rows <= 4096u ? 4u : n_rows <= 8192u ? 2u : 1u, by_steps = (g.en + 1u) / 2u;
  return by_steps < most ? by_steps : most;
}

// Lanes on the cells of a word, walking n; what is decided is a ballot and stays in scalar registers (lane t of a
// vector register keeps step t's word for the store).
constexpr int kRowSteps = 8;              // steps whose reads are in flight together

__global__ __launch_bounds__(256) void row_heads_kernel(const RowGeo g, const RowBufs B, const uint64_t* __restrict__ cost,
                                                        const uint16_t* __restrict__ arg, const u64* __restrict__ fit,
                                                        const uint32_t* __restrict__ sizes) {
  const uint32_t lane = threadIdx.x & 63u, n_rows = B.tot[kRowsTotal];
  RowWords W;
  if (!row_words(g, B, W)) return;
  const uint32_t size_n = lane < g.en ? axis_sizes(g, sizes, 3)[lane] : 1u;
  for (uint32_t row = first_row(); row < n_rows; row += gridDim.x * 4u) {
    const WaveRow r(B, row);
    const u64 words = lane < g.en ? fit[((size_t)(r.shape0 + lane) << g.lg_nw) + r.w] : 0ull;
    const u64 live = __ballot(words != 0);
    const uint32_t n_live = live ? 64u - (uint32_t)__builtin_clzll(live) : 0u;     // from there on every cell is (INF, NONE)
    u64 hd = lane == 0 ? ~0ull : 0ull, hc = hd, pinf = ~0ull;
    uint64_t pc = kInf;
    uint32_t pa = kNone, ps = 1;
    for (uint32_t t0 = 0; t0 < n_live; t0 += kRowSteps) {
      uint64_t c[kRowSteps];
      uint32_t a[kRowSteps];
#pragma unroll
      for (int u = 0; u < kRowSteps; u++) {
        const uint32_t t = t0 + u < n_live ? t0 + u : n_live - 1u;
        c[u] = kInf; a[u] = kNone;
        if (in_mask(lane64(words, t))) {
          const size_t at = (size_t)(r.shape0 + t) * g.G + r.w * 64u;
          c[u] = (cost + at)[lane];
          a[u] = (arg + at)[lane];
        }
      }
#pragma unroll
      for (int u = 0; u < kRowSteps; u++) {
        const uint32_t t = t0 + u;
        if (t >= n_live) break;
        const u64 inf = infinite(c[u]);
        const uint32_t s = (uint32_t)__builtin_amdgcn_readlane((int)size_n, (int)t);
        if (t) {
          put_lane64(hd, __ballot(a[u] != pa), t);
          put_lane64(hc, ~equal_costs(c[u], s, inf, pc, ps, pinf), t);
        }
        pc = c[u]; pa = a[u]; ps = s; pinf = inf;
      }
    }
    if (n_live && n_live < g.en) {
      put_lane64(hd, __ballot(pa != kNone), n_live);
      put_lane64(hc, ~pinf, n_live);
    }
    if (lane < g.en) {
      const size_t at = (size_t)r.row * g.en + lane;
      W.H[0][at] = hd;
      W.H[1][at] = hc;
    }
  }
}

// Lane i gets lane i + d's value (any value where there is none).
__device__ __forceinline__ u64 above64(u64 x, uint32_t d) {
  const int from = (int)((threadIdx.x & 63u) + d);
  return (u64)(uint32_t)__shfl((int)(uint32_t)(x >> 32), from, 64) << 32 | (uint32_t)__shfl((int)(uint32_t)x, from, 64);
}

// Heads of row 0 (the wave's) and of a row before it whose runs are equally long: the next head above them, if any, is
// the same step in both rows.  Lane n has the words of step n; seen from the far end a step settles that where it has
// heads (both), passes it on where it has none (a prefix computation over the lanes).
__device__ __forceinline__ u64 same_runs(u64 h, u64 h1, uint32_t en) {
  const uint32_t lane = threadIdx.x & 63u;
  const u64 both = h & h1, used = __ballot((h | h1) != 0 && lane < en);
  en = used ? 64u - (uint32_t)__builtin_clzll(used) : 0u;           // (no heads further on)
  u64 hit = lane < en ? both : ~0ull, pass = lane < en ? ~(h | h1) : 0ull;
  for (uint32_t d = 1; d < en; d <<= 1) {
    u64 nh = above64(hit, d), np = above64(pass, d);
    if (lane + d >= 64u) { nh = ~0ull; np = 0; }
    hit |= pass & nh;
    pass &= np;
  }
  u64 above = above64(hit, 1), open = above64(pass, 1);
  if (lane == 63u) { above = ~0ull; open = 0; }
  return both & (above | open);
}

constexpr int kAgreeSteps = 4;

template <int NX>
__global__ __launch_bounds__(256) void row_agree_kernel(const RowGeo g, const RowBufs B, const uint64_t* __restrict__ cost,
                                                        const uint16_t* __restrict__ arg, const uint32_t* __restrict__ sizes) {
  const uint32_t lane = threadIdx.x & 63u, n_rows = B.tot[kRowsTotal];
  RowWords W;
  if (!row_words(g, B, W)) return;
  const uint32_t parts = row_parts(g, n_rows), each = (g.en + parts - 1u) / parts;
  for (uint32_t i = first_row(); i < parts * n_rows; i += gridDim.x * 4u) {
    const uint32_t row = i / parts;
    const bool mine = lane < g.en && lane / each == i % parts;
    const WaveRow r(B, row);
    // rows 1 to 3: the ones before on k, m, b
    const uint32_t back[4] = {0, g.en, g.ek * g.en, g.em * g.ek * g.en};
    const uint32_t before[4] = {row, row - 1u, r.m_before, r.b_before};
    const bool has[4] = {true, r.k > 0, r.m > 0, r.b > 0};
    const uint32_t *size_k = axis_sizes(g, sizes, 2) + r.k, *size_m = axis_sizes(g, sizes, 1) + r.m, *size_b = axis_sizes(g, sizes, 0) + r.b;
    const uint32_t sz[4] = {1u, size_k[0], size_m[0], size_b[0]};
    const uint32_t sz1[4] = {1u, r.k ? size_k[-1] : 1u, r.m ? size_m[-1] : 1u, r.b ? size_b[-1] : 1u};
    const size_t at = (size_t)r.row * g.en + lane;
    u64 h[2], cand[2][4];
#pragma unroll
    for (int l = 0; l < 2; l++) h[l] = lane < g.en ? W.H[l][at] : 0ull;
#pragma unroll
    for (int x = 1; x < NX; x++) {
      const bool kept = before[x] != kNoRow;
      const size_t at1 = (size_t)(kept ? before[x] : row) * g.en + lane;
#pragma unroll
      for (int l = 0; l < 2; l++) {
        cand[l][x] = 0;
        if (!has[x]) continue;
        const u64 h1 = lane < g.en ? (kept ? W.H[l][at1] : gone_word(lane)) : 0ull;
        cand[l][x] = same_runs(h[l], h1, g.en);
        if (!mine) cand[l][x] = 0;
      }
    }
    u64 any = 0;
#pragma unroll
    for (int x = 1; x < NX; x++) any |= cand[0][x] | cand[1][x];
    u64 todo = __ballot(any != 0);
    while (todo) {
      uint32_t t[kAgreeSteps];
      uint64_t c[NX][kAgreeSteps];
      uint32_t a[NX][kAgreeSteps];
      u64 m[2][NX][kAgreeSteps];
      int n = 0;
#pragma unroll
      for (int u = 0; u < kAgreeSteps; u++) {
        t[u] = todo ? (uint32_t)__builtin_ctzll(todo) : 0u;
        const bool on = todo != 0;
        n += on ? 1 : 0;
        todo &= todo - 1;                 // 0 stays 0
        const size_t cell = (size_t)(r.shape0 + t[u]) * g.G + r.w * 64u;
        u64 md = 0, mc = 0;
#pragma unroll
        for (int x = 1; x < NX; x++) {
          m[0][x][u] = on ? lane64(cand[0][x], t[u]) : 0ull; m[1][x][u] = on ? lane64(cand[1][x], t[u]) : 0ull;
          md |= m[0][x][u]; mc |= m[1][x][u];
          const size_t cell1 = cell - (size_t)back[x] * g.G;
          c[x][u] = 0; a[x][u] = 0;
          if (in_mask(m[1][x][u])) c[x][u] = (cost + cell1)[lane];
          if (in_mask(m[0][x][u])) a[x][u] = (arg + cell1)[lane];
        }
        c[0][u] = 0; a[0][u] = 0;
        if (in_mask(mc)) c[0][u] = (cost + cell)[lane];
        if (in_mask(md)) a[0][u] = (arg + cell)[lane];
      }
#pragma unroll
      for (int u = 0; u < kAgreeSteps; u++) {
        if (u >= n) break;
        const u64 inf0 = infinite(c[0][u]);
#pragma unroll
        for (int x = 1; x < NX; x++) {
          if (m[0][x][u]) put_lane64(cand[0][x], m[0][x][u] & __ballot(a[0][u] == a[x][u]), t[u]);
          if (m[1][x][u]) put_lane64(cand[1][x], m[1][x][u] & equal_costs(c[0][u], sz[x], inf0, c[x][u], sz1[x], infinite(c[x][u])), t[u]);
        }
      }
    }
    if (mine) {
#pragma unroll
      for (int l = 0; l < 2; l++) {
        W.Fk[l][at] = cand[l][1];
        if (g.em > 1) W.Fm[l][at] = cand[l][2];                     // (that agree: the kernels below decide)
        if (NX > 3) W.Fb[l][at] = cand[l][NX - 1];
      }
    }
  }
}

// A lane per (plane, n), bits = cells, walking k from the far end: heads of rows m and m - 1 that agree are folded if
// their chains along k are equally long (`same`).  Rows are read kFoldRows at a time: the walk is a chain of a
// few word operations, the reads are not.
constexpr int kFoldRows = 8;

__global__ __launch_bounds__(256) void row_fold_m_kernel(const RowGeo g, const RowBufs B) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x, l = blockIdx.y;
  const uint32_t p = i / g.en, n = i - p * g.en;
  if (p >= g.n_planes) return;
  RowWords W;
  if (!row_words(g, B, W)) return;
  if ((p >> g.lg_nw) % g.em == 0) return;                     // (m = 0 agrees with nothing)
  const uint32_t K = B.rows[p], K1 = B.rows[p - g.nw];
  const size_t at0 = (size_t)B.first[p] * g.en + n, at1 = (size_t)B.first[p - g.nw] * g.en + n;
  const u64* __restrict__ H = l ? W.H[1] : W.H[0];
  const u64* __restrict__ Fk = l ? W.Fk[1] : W.Fk[0];
  u64* __restrict__ Fm = l ? W.Fm[1] : W.Fm[0];
  const u64 gone = gone_word(n);
  u64 same = ~0ull;
  for (int k0 = (int)(K > K1 ? K : K1) - 1; k0 >= 0; k0 -= kFoldRows) {
    u64 f[kFoldRows], f1[kFoldRows], left[kFoldRows];
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {       // (rows that are not there: another one is read and not used)
      const uint32_t k = k0 - u > 0 ? (uint32_t)(k0 - u) : 0u;
      const size_t j = at0 + (size_t)(k < K ? k : K - 1u) * g.en, j1 = at1 + (size_t)(k < K1 ? k : K1 - 1u) * g.en;
      const u64 own = Fk[j], other = Fk[j1];
      left[u] = Fm[j] & H[j] & H[j1];
      f[u] = k < K ? own : gone;
      f1[u] = k < K1 ? other : gone;
    }
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      const int k = k0 - u;
      if (k >= 0 && (uint32_t)k < K) Fm[at0 + (size_t)k * g.en] = (uint32_t)k < K1 ? left[u] & ~f[u] & ~f1[u] & same : 0ull;
      same = ~(f[u] ^ f1[u]) & (~f[u] | same);
    }
  }
}

// The same for b in two steps: chains along k compared (a lane per plane and n), then along m (a lane per b, place, k, n).
__global__ __launch_bounds__(256) void row_fold_b_k_kernel(const RowGeo g, const RowBufs B) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x, l = blockIdx.y;
  const uint32_t p = i / g.en, n = i - p * g.en, bstep = g.em * g.nw;
  if (p >= g.n_planes || p < bstep) return;                  // (b = 0 agrees with nothing)
  RowWords W;
  if (!row_words(g, B, W)) return;
  const uint32_t K = B.rows[p], K1 = B.rows[p - bstep];
  const size_t at0 = (size_t)B.first[p] * g.en + n, at1 = (size_t)B.first[p - bstep] * g.en + n;
  const u64* __restrict__ H = l ? W.H[1] : W.H[0];
  const u64* __restrict__ Fk = l ? W.Fk[1] : W.Fk[0];
  const u64* __restrict__ Fm = l ? W.Fm[1] : W.Fm[0];
  u64* __restrict__ Fb = l ? W.Fb[1] : W.Fb[0];
  const bool has_m = g.em > 1;
  const u64 gone = gone_word(n);
  u64 same = ~0ull;
  for (int k0 = (int)(K > K1 ? K : K1) - 1; k0 >= 0; k0 -= kFoldRows) {
    u64 f[kFoldRows], f1[kFoldRows], left[kFoldRows];
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      const uint32_t k = k0 - u > 0 ? (uint32_t)(k0 - u) : 0u;
      const size_t j = at0 + (size_t)(k < K ? k : K - 1u) * g.en, j1 = at1 + (size_t)(k < K1 ? k : K1 - 1u) * g.en;
      const u64 own = Fk[j], other = Fk[j1];
      left[u] = Fb[j] & H[j] & H[j1];
      if (has_m) left[u] &= ~(Fm[j] | Fm[j1]);
      f[u] = k < K ? own : gone;
      f1[u] = k < K1 ? other : gone;
    }
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      const int k = k0 - u;
      if (k >= 0 && (uint32_t)k < K) Fb[at0 + (size_t)k * g.en] = (uint32_t)k < K1 ? left[u] & ~f[u] & ~f1[u] & same : 0ull;
      same = ~(f[u] ^ f1[u]) & (~f[u] | same);
    }
  }
}

__global__ __launch_bounds__(256) void row_fold_b_m_kernel(const RowGeo g, const RowBufs B) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x, l = blockIdx.y;
  const uint32_t n = i % g.en, q = i / g.en, k = q % g.ek, bw = q / g.ek, w = bw & (g.nw - 1u), b = bw >> g.lg_nw;
  if (b >= g.eb || b == 0) return;
  RowWords W;
  if (!row_words(g, B, W)) return;
  const u64* __restrict__ Fm = l ? W.Fm[1] : W.Fm[0];
  u64* __restrict__ Fb = l ? W.Fb[1] : W.Fb[0];
  u64 same = ~0ull;
  for (int m0 = (int)g.em - 1; m0 >= 0; m0 -= kFoldRows) {
    u64 f[kFoldRows], f1[kFoldRows], fold[kFoldRows];
    size_t at[kFoldRows];
    bool own[kFoldRows];
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {       // (rows that are not there: another one is read and not used)
      const int m = m0 - u;
      const uint32_t p = ((b * g.em + (uint32_t)(m > 0 ? m : 0)) << g.lg_nw) + w, p1 = p - g.em * g.nw;
      const uint32_t K = B.rows[p], K1 = B.rows[p1];
      own[u] = m >= 0 && k < K;
      const bool other = m >= 0 && k < K1;
      at[u] = ((size_t)B.first[p] + (k < K ? k : K - 1u)) * g.en + n;
      const size_t at1 = ((size_t)B.first[p1] + (k < K1 ? k : K1 - 1u)) * g.en + n;
      f[u] = f1[u] = 0;
      if (g.em > 1) { f[u] = Fm[at[u]]; f1[u] = Fm[at1]; }
      fold[u] = Fb[at[u]];
      f[u] = own[u] ? f[u] : 0ull;
      f1[u] = other ? f1[u] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      if (own[u]) Fb[at[u]] = fold[u] & same;
      same = ~(f[u] ^ f1[u]) & (~f[u] | same);
    }
  }
}

// The same for chains longer than a wave: the lanes on 64 steps of a chain, `same` by a prefix computation over them.  A
// lane per chain reads a place of its own with every load there, and there are few chains.  3 sizes along b, 4 along m and n,
// all to 255 along k: row_fold_b_k_kernel 140 us, this 6, the solve 761 -> 574; all to 255 along m, 4 along k:
// row_fold_b_m_kernel 99 us, this 9, the solve 656 -> 560.  (box by box 708 and 697)
// f, f1: the folds of the lane's step; same: of the step behind the 64, then of their first.  Returns that of the step behind the lane's.
__device__ __forceinline__ u64 same_behind(u64 f, u64 f1, u64& same) {
  const uint32_t lane = threadIdx.x & 63u;
  u64 hit = ~(f | f1), pass = f & f1;                               // `same` of a step is hit | pass & the next one's
#pragma unroll
  for (uint32_t d = 1; d < 64; d <<= 1) {
    const u64 nh = above64(hit, d), np = above64(pass, d);
    hit |= lane + d < 64u ? pass & nh : 0ull;
    pass &= lane + d < 64u ? np : ~0ull;
  }
  const u64 nh = above64(hit, 1), np = above64(pass, 1), behind = lane < 63u ? nh | (np & same) : same;
  same = lane64(hit, 0) | (lane64(pass, 0) & same);
  return behind;
}

// Chains along k, for m or for b's first step: a wave per (plane, n).
__global__ __launch_bounds__(256) void row_fold_long_k_kernel(const RowGeo g, const RowBufs B, uint32_t along_b) {
  const uint32_t lane = threadIdx.x & 63u, i = first_row(), l = blockIdx.y;
  const uint32_t p = i / g.en, n = i - p * g.en, step = along_b ? g.em * g.nw : g.nw;
  if (p >= g.n_planes) return;
  RowWords W;
  if (!row_words(g, B, W)) return;
  if (along_b ? p < step : (p >> g.lg_nw) % g.em == 0) return;      // (the first along the axis agrees with nothing)
  const uint32_t K = B.rows[p], K1 = B.rows[p - step];
  const size_t at0 = (size_t)B.first[p] * g.en + n, at1 = (size_t)B.first[p - step] * g.en + n;
  const u64* __restrict__ H = l ? W.H[1] : W.H[0];
  const u64* __restrict__ Fk = l ? W.Fk[1] : W.Fk[0];
  const u64* Fm = l ? W.Fm[1] : W.Fm[0];
  u64* F = along_b ? (l ? W.Fb[1] : W.Fb[0]) : (l ? W.Fm[1] : W.Fm[0]);
  const bool not_m = along_b && g.em > 1;
  const u64 gone = gone_word(n);
  u64 same = ~0ull;
  for (int k0 = (int)(((K > K1 ? K : K1) - 1u) & ~63u); k0 >= 0; k0 -= 64) {
    const uint32_t k = (uint32_t)k0 + lane;     // (rows that are not there: another one is read and not used)
    const size_t j = at0 + (size_t)(k < K ? k : K - 1u) * g.en, j1 = at1 + (size_t)(k < K1 ? k : K1 - 1u) * g.en;
    const u64 own = Fk[j], other = Fk[j1];
    u64 left = F[j] & H[j] & H[j1];
    if (not_m) left &= ~(Fm[j] | Fm[j1]);
    const u64 f = k < K ? own : gone, f1 = k < K1 ? other : gone, behind = same_behind(f, f1, same);
    if (k < K) F[j] = k < K1 ? left & ~f & ~f1 & behind : 0ull;
  }
}

// Chains along m, for b's second step: a wave per (b, place, k, n).
__global__ __launch_bounds__(256) void row_fold_long_m_kernel(const RowGeo g, const RowBufs B) {
  const uint32_t lane = threadIdx.x & 63u, i = first_row(), l = blockIdx.y;
  const uint32_t n = i % g.en, q = i / g.en, k = q % g.ek, bw = q / g.ek, w = bw & (g.nw - 1u), b = bw >> g.lg_nw;
  if (b >= g.eb || b == 0) return;
  RowWords W;
  if (!row_words(g, B, W)) return;
  const u64* __restrict__ Fm = l ? W.Fm[1] : W.Fm[0];
  u64* __restrict__ Fb = l ? W.Fb[1] : W.Fb[0];
  u64 same = ~0ull;
  for (int m0 = (int)((g.em - 1u) & ~63u); m0 >= 0; m0 -= 64) {
    const uint32_t m = (uint32_t)m0 + lane, p = ((b * g.em + (m < g.em ? m : 0u)) << g.lg_nw) + w, p1 = p - g.em * g.nw;
    const uint32_t K = B.rows[p], K1 = B.rows[p1];
    const bool own = m < g.em && k < K, other = m < g.em && k < K1;
    const size_t at = ((size_t)B.first[p] + (k < K ? k : K - 1u)) * g.en + n, at1 = ((size_t)B.first[p1] + (k < K1 ? k : K1 - 1u)) * g.en + n;
    const u64 f = Fm[at], f1 = Fm[at1], fold = Fb[at], behind = same_behind(own ? f : 0ull, other ? f1 : 0ull, same);
    if (own) Fb[at] = fold & behind;
  }
}

// A lane per word: the heads left of both lists, and those of them that some step or row after theirs was folded into.
__global__ __launch_bounds__(256) void row_left_kernel(const RowGeo g, const RowBufs B) {
  RowWords W;
  if (!row_words(g, B, W)) return;
  const uint32_t n_words = B.tot[kRowsTotal] * g.en;
  for (uint32_t at = blockIdx.x * 256u + threadIdx.x; at < n_words; at += gridDim.x * 256u) {
    const uint32_t row = at / g.en, n = at - row * g.en;
    const RowInfo* __restrict__ info = (const RowInfo*)B.info + row;
    const uint32_t k = info->k, kept = info->kept, m_after = info->m_after, b_after = info->b_after;
    // the rows after it on m and b, where they are kept (else the row itself, and not used)
    const size_t at_m = m_after != kNoRow ? (size_t)m_after * g.en + n : at, at_b = b_after != kNoRow ? (size_t)b_after * g.en + n : at;
    const size_t at_k = k + 1u < kept ? (size_t)at + g.en : at, at_n = n + 1u < g.en ? (size_t)at + 1 : at;
    const u64 past_k = k + 1u < g.ek ? gone_word(n) : 0ull;
#pragma unroll
    for (int l = 0; l < 2; l++) {
      const u64 up = W.H[l][at_n], k1 = W.Fk[l][at_k];
      u64 t = W.H[l][at] & ~W.Fk[l][at], more = (n + 1u < g.en ? ~up : 0ull) | (k + 1u < kept ? k1 : past_k);
      if (g.em > 1) { const u64 m1 = W.Fm[l][at_m]; t &= ~W.Fm[l][at]; more |= m_after != kNoRow ? m1 : 0ull; }
      if (g.eb > 1) { const u64 b1 = W.Fb[l][at_b]; t &= ~W.Fb[l][at]; more |= b_after != kNoRow ? b1 : 0ull; }
      const size_t at_l = (l ? (size_t)n_words : 0) + at;
      W.T[at_l] = t;
      W.N[at_l] = t & more;
    }
  }
}

// ---------------------------------------------------------------- extents on the size axes
// A wave per row, the words with heads in N: the words further on along an axis are gathered, a lane each, and only the
// steps at which some chain ends are looked at.
__global__ __launch_bounds__(256) void row_extent_kernel(const RowGeo g, const RowBufs B) {
  const uint32_t lane = threadIdx.x & 63u, n_rows = B.tot[kRowsTotal];
  RowWords W;
  if (!row_words(g, B, W, true)) return;
  const uint32_t parts = row_parts(g, n_rows), each = (g.en + parts - 1u) / parts;
  for (uint32_t ip = first_row(); ip < 2u * parts * n_rows; ip += gridDim.x * 4u) {
    const uint32_t i = ip / parts, l = i < n_rows ? 1u : 0u;
    const WaveRow r(B, l ? i : i - n_rows);
    const uint32_t plane = r.plane, k = r.k, row = r.row, b = r.b, m = r.m, K = r.kept;
    const u64* Hl = l ? W.H[1] : W.H[0];
    const u64* Fk = l ? W.Fk[1] : W.Fk[0];
    const u64* Fm = l ? W.Fm[1] : W.Fm[0];
    const u64* Fb = l ? W.Fb[1] : W.Fb[0];
    const size_t at = (size_t)row * g.en + lane, at_t = (l ? (size_t)B.tot[kRowsTotal] * g.en : 0) + at;
    const bool mine = lane < g.en;
    const u64 t = mine ? W.N[at_t] : 0ull;
    u64 todo = __ballot(t != 0 && lane / each == ip % parts);
    if (!todo) continue;
    const u64 h = mine ? Hl[at] : ~0ull;
    const uint32_t rank = mine ? W.rank[at_t].x : 0u;
    // word n of row k + c (m + c, b + c): its heads folded into the row before
    auto word_k = [&](uint32_t c, uint32_t n) -> u64 { return k + c < K ? Fk[(size_t)(row + c) * g.en + n] : k + c < g.ek ? gone_word(n) : 0ull; };
    auto word_m = [&](uint32_t c, uint32_t n) -> u64 {
      if (m + c >= g.em) return 0;
      const uint32_t p = plane + c * g.nw;
      return k < B.rows[p] ? Fm[(size_t)(B.first[p] + k) * g.en + n] : 0ull;
    };
    auto word_b = [&](uint32_t c, uint32_t n) -> u64 {
      if (b + c >= g.eb) return 0;
      const uint32_t p = plane + c * g.em * g.nw;
      return k < B.rows[p] ? Fb[(size_t)(B.first[p] + k) * g.en + n] : 0ull;
    };
    const uint32_t n_up = lane + 1u < g.en ? lane + 1u : lane;
    const u64 h_up = (u64)__shfl((uint32_t)(h >> 32), n_up, 64) << 32 | (uint32_t)__shfl((uint32_t)h, n_up, 64);
    const u64 long_n = lane + 1u < g.en ? t & ~h_up : 0ull;
    const u64 long_k = mine ? t & word_k(1, lane) : 0ull;
    const u64 long_m = mine && r.m_after != kNoRow ? t & Fm[(size_t)r.m_after * g.en + lane] : 0ull;
    const u64 long_b = mine && r.b_after != kNoRow ? t & Fb[(size_t)r.b_after * g.en + lane] : 0ull;
    const u64 has_n = __ballot(long_n != 0), has_k = __ballot(long_k != 0), has_m = __ballot(long_m != 0), has_b = __ballot(long_b != 0);
    // cells of `cur` have extent 2 or more; word(c, n): the chain goes on to step c
    auto walk = [&](u64 cur, uint32_t n, uint32_t shift, uint32_t& e, u64 on, auto&& word) {      // on: word(2 + lane, n)
      for (uint32_t c0 = 2; cur; c0 += 64) {
        if (c0 > 2) on = word(c0 + lane, n);
        for (;;) {
          const u64 ends = __ballot((cur & ~on) != 0);
          if (!ends) break;
          const uint32_t c = (uint32_t)__builtin_ctzll(ends);
          const u64 on_c = lane64(on, c);
          if (in_mask(cur & ~on_c)) e += (c0 + c - 1u) << shift;
          cur &= on_c;
          if (!cur) break;
        }
      }
    };
    while (todo) {
      const uint32_t n = (uint32_t)__builtin_ctzll(todo);
      todo &= todo - 1;
      const u64 tn = lane64(t, n);
      const uint32_t at_rank = (uint32_t)__builtin_amdgcn_readlane((int)rank, (int)n) + below(tn);
      uint32_t e = 0x01010101u;                                   // a byte per size axis, in the coordinates' order
      const bool go_k = (has_k >> n) & 1ull, go_m = (has_m >> n) & 1ull, go_b = (has_b >> n) & 1ull;
      const u64 on_k = go_k ? word_k(2u + lane, n) : 0ull, on_m = go_m ? word_m(2u + lane, n) : 0ull, on_b = go_b ? word_b(2u + lane, n) : 0ull;
      if ((has_n >> n) & 1ull) {
        u64 cur = lane64(long_n, n);
        while (cur) {
          const u64 ends = __ballot(lane > n && ((h & cur) != 0 || lane >= g.en));
          const uint32_t c = ends ? (uint32_t)__builtin_ctzll(ends) : g.en;      // (64 steps: no lane is left to end the list)
          const u64 gone = c < g.en ? cur & lane64(h, c) : cur;
          if (in_mask(gone)) e += (c - n - 1u) << (8u * g.axis[3]);
          cur &= ~gone;
        }
      }
      if (go_k) walk(lane64(long_k, n), n, 8u * g.axis[2], e, on_k, word_k);
      if (go_m) walk(lane64(long_m, n), n, 8u * g.axis[1], e, on_m, word_m);
      if (go_b) walk(lane64(long_b, n), n, 8u * g.axis[0], e, on_b, word_b);
      if (in_mask(tn)) W.ext[at_rank] = e;
    }
  }
}

// ---------------------------------------------------------------- the axes inside a shape
// Lane i gets lane i + 2^bit's value, for lanes whose field at that bit is not at its end (row_shl: inside 16
// lanes, as far as a field of two bits at bit 2 goes).
// bit is a constant of an unrolled loop.
__device__ __forceinline__ uint32_t step_above(int bit, uint32_t x) {
  switch (bit) {
    case 0: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x101, 0xF, 0xF, true);
    case 1: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x102, 0xF, 0xF, true);
    case 2: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x104, 0xF, 0xF, true);
    default: return (uint32_t)__shfl((int)x, (int)((threadIdx.x & 63u) + (1u << bit)), 64);
  }
}
// The cells of a word whose field of `bits` bits at bit b is not at its end.
__device__ __forceinline__ u64 not_last(uint32_t b, bool two) {
  const u64 one = b == 0 ? 0x5555555555555555ull : b == 1 ? 0x3333333333333333ull : b == 2 ? 0x0F0F0F0F0F0F0F0Full : b == 3 ? 0x00FF00FF00FF00FFull
                : b == 4 ? 0x0000FFFF0000FFFFull : 0x00000000FFFFFFFFull;
  const u64 above = b == 0 ? 0x3333333333333333ull : b == 1 ? 0x0F0F0F0F0F0F0F0Full : b == 2 ? 0x00FF00FF00FF00FFull : b == 3 ? 0x0000FFFF0000FFFFull : 0x00000000FFFFFFFFull;
  return two ? one | above : one;
}

// Where `agree` has the words of an axis: level axis q, or the field that starts at bit b.
__device__ __forceinline__ u64* agree_level(const RowGeo& g, const RowWords& W, size_t both, uint32_t q) { return W.agree + both * q; }
__device__ __forceinline__ bool field_at(const RowGeo& g, uint32_t b) { return (g.var_first >> b) & 1u; }
__device__ __forceinline__ u64* agree_field(const RowGeo& g, const RowWords& W, size_t both, uint32_t b) {
  return W.agree + both * (g.n_levels + (uint32_t)__popc(g.var_first & ((1u << b) - 1u)));
}
__device__ __forceinline__ size_t agree_stride(const RowGeo& g, uint32_t n_rows) { return 2 * (size_t)n_rows * g.en; }

// Level axis q (in merge order) is the bits [LV + 2 q, LV + 2 q + 2) of a cell's place in the shape: inside a word, or the
// next word's row (the one step further of 32 cells runs over two words).
constexpr int kInnerSteps = 2;            // words whose values are read together

template <bool COST, int LV>
__device__ __forceinline__ void row_inner(const RowGeo& g, const RowBufs& B, const RowWords& W, uint32_t n_rows, uint32_t row, uint32_t part, uint32_t parts,
                                          const uint64_t* __restrict__ cost, const uint16_t* __restrict__ arg) {
  constexpr int kLevels = (int)kRowLevels;
  const uint32_t lane = threadIdx.x & 63u;
  const WaveRow r(B, row);
  const size_t list = COST ? (size_t)n_rows * g.en : 0, at = list + (size_t)row * g.en + lane;
  const uint32_t each = (g.en + parts - 1u) / parts;
  const bool mine = lane < g.en && lane / each == part;
  const u64 T = mine ? W.T[at] : 0ull;
  if (!__ballot(T != 0)) return;
  const u64 N = T ? W.N[at] : 0ull;
  const uint32_t rank = N ? W.rank[at].x : 0u;
  u64 lev[kLevels], var[LV ? LV : 1];
  size_t next[kLevels];                    // the next word's place, where the axis leaves the word
#pragma unroll
  for (int q = 0; q < kLevels; q++) {
    lev[q] = 0; next[q] = at;
    if ((uint32_t)q >= g.n_levels) continue;
    const int sh = LV + 2 * q;
    if (sh >= 5) {
      const bool kept = r.next[q] != kNoRow;
      if (kept) next[q] = list + (size_t)r.next[q] * g.en + lane;
      const u64 t1 = kept && mine ? W.T[next[q]] : 0ull, n1 = kept && mine ? W.N[next[q]] : 0ull;
      if (sh >= 6) lev[q] = T & t1 & ~(N ^ n1);
      else lev[q] = T & (T >> 32 | t1 << 32) & ~(N ^ (N >> 32 | n1 << 32)) & (r.w & 1u ? 0xFFFFFFFFull : ~0ull);
    } else {
      lev[q] = T & T >> (1 << (sh < 6 ? sh : 0)) & ~(N ^ N >> (1 << (sh < 6 ? sh : 0))) & not_last(sh, true);
    }
  }
#pragma unroll
  for (int b = 0; b < LV; b++)
    var[b] = field_at(g, b) ? T & T >> (1 << b) & ~(N ^ N >> (1 << b)) & not_last(b, (g.var_two >> b) & 1u) : 0ull;

  // ---- values, the lanes on a word's cells ----
  u64 pairs = 0;
#pragma unroll
  for (int q = 0; q < kLevels; q++) pairs |= lev[q];
#pragma unroll
  for (int b = 0; b < LV; b++) pairs |= var[b];
  for (u64 todo = __ballot(pairs != 0); todo;) {
    uint32_t t[kInnerSteps];
    uint64_t v[kInnerSteps], v2[kInnerSteps][kLevels];
    u64 m[kInnerSteps][kLevels];
    bool some[kInnerSteps];
#pragma unroll
    for (int u = 0; u < kInnerSteps; u++) {
      some[u] = todo != 0;
      t[u] = todo ? (uint32_t)__builtin_ctzll(todo) : 0u;
      todo &= todo - 1;                 // 0 stays 0
      const size_t cell0 = (size_t)(r.shape0 + t[u]) * g.G + r.w * 64u;
      const uint64_t* c64 = cost + cell0;
      const uint16_t* a16 = arg + cell0;
      const u64 tw = some[u] ? lane64(T, t[u]) : 0ull;
      v[u] = 0;
      if (in_mask(tw)) v[u] = COST ? c64[lane] : (uint64_t)a16[lane];
#pragma unroll
      for (int q = 0; q < kLevels; q++) {
        m[u][q] = 0; v2[u][q] = 0;
        if ((uint32_t)q >= g.n_levels) continue;
        const int sh = LV + 2 * q;
        m[u][q] = some[u] ? lane64(lev[q], t[u]) : 0ull;
        if (sh >= 5 && in_mask(m[u][q])) v2[u][q] = COST ? c64[(1u << sh) + lane] : (uint64_t)a16[(1u << sh) + lane];
      }
    }
#pragma unroll
    for (int u = 0; u < kInnerSteps; u++) {
      if (!some[u]) break;
#pragma unroll
      for (int q = 0; q < kLevels; q++) {
        const int sh = LV + 2 * q;
        if ((uint32_t)q >= g.n_levels || !m[u][q]) continue;
        if (sh < 5) {
          v2[u][q] = step_above(sh, (uint32_t)v[u]);
          if (COST) v2[u][q] |= (uint64_t)step_above(sh, (uint32_t)(v[u] >> 32)) << 32;
        }
        put_lane64(lev[q], m[u][q] & __ballot(v[u] == v2[u][q]), t[u]);
      }
#pragma unroll
      for (int b = 0; b < LV; b++) {
        const u64 mb = lane64(var[b], t[u]);
        if (!mb) continue;
        uint64_t vb = step_above(b, (uint32_t)v[u]);
        if (COST) vb |= (uint64_t)step_above(b, (uint32_t)(v[u] >> 32)) << 32;
        put_lane64(var[b], mb & __ballot(v[u] == vb), t[u]);
      }
    }
  }
  // ---- and the size extents, where both heads have some above 1 ----
  pairs = 0;
#pragma unroll
  for (int q = 0; q < kLevels; q++) pairs |= lev[q];
#pragma unroll
  for (int b = 0; b < LV; b++) pairs |= var[b];
  for (u64 todo = __ballot((pairs & N) != 0); todo; todo &= todo - 1) {
    const uint32_t t = (uint32_t)__builtin_ctzll(todo);
    const u64 nw = lane64(N, t);
    uint32_t e = 0;
    if (in_mask(nw)) e = W.ext[(uint32_t)__builtin_amdgcn_readlane((int)rank, (int)t) + below(nw)];
#pragma unroll
    for (int q = 0; q < kLevels; q++) {
      if ((uint32_t)q >= g.n_levels) continue;
      const int sh = LV + 2 * q;
      const u64 m = lane64(lev[q], t);
      if (!(m & nw)) continue;
      uint32_t e2 = 0;
      if (sh >= 5) {
        const size_t o = (size_t)lane64(next[q], t);
        const u64 n1 = W.N[o];
        const uint32_t rank1 = W.rank[o].x;
        if (sh >= 6) {
          if (in_mask(m & nw)) e2 = W.ext[rank1 + below(n1)];
        } else {
          e2 = (uint32_t)__shfl((int)e, (int)(lane + 32u), 64);
          if (lane >= 32u && in_mask(m & nw)) e2 = W.ext[rank1 + __popc((uint32_t)n1 & ((1u << (lane & 31u)) - 1u))];
        }
      } else {
        e2 = (uint32_t)__shfl((int)e, (int)(lane + (1u << (sh < 6 ? sh : 0))), 64);
      }
      put_lane64(lev[q], m & (~nw | __ballot(e == e2)), t);
    }
#pragma unroll
    for (int b = 0; b < LV; b++) {
      const u64 m = lane64(var[b], t);
      if (!(m & nw)) continue;
      const uint32_t e2 = (uint32_t)__shfl((int)e, (int)(lane + (1u << b)), 64);
      put_lane64(var[b], m & (~nw | __ballot(e == e2)), t);
    }
  }
  if (T) {
    const size_t both = agree_stride(g, n_rows);
#pragma unroll
    for (int q = 0; q < kLevels; q++) if ((uint32_t)q < g.n_levels) agree_level(g, W, both, q)[at] = lev[q];
#pragma unroll
    for (int b = 0; b < LV; b++) if (field_at(g, b)) agree_field(g, W, both, b)[at] = var[b];
  }
}

template <int LV>
__global__ __launch_bounds__(256) void row_inner_kernel(const RowGeo g, const RowBufs B, const uint64_t* __restrict__ cost, const uint16_t* __restrict__ arg) {
  RowWords W;
  if (!row_words(g, B, W, true)) return;
  const uint32_t n_rows = B.tot[kRowsTotal], parts = row_parts(g, n_rows);
  for (uint32_t i = first_row(); i < 2u * parts * n_rows; i += gridDim.x * 4u) {
    const uint32_t part = i % parts, row = i / parts;
    if (row < n_rows) row_inner<true, LV>(g, B, W, n_rows, row, part, parts, cost, arg);
    else row_inner<false, LV>(g, B, W, n_rows, row - n_rows, part, parts, cost, arg);
  }
}

constexpr uint32_t kMergeWords = 256;      // words of a batch, a lane each
constexpr uint32_t kNoWord = kMergeWords;  // LDS place of a word without heads
constexpr uint32_t kGroupWords = 2048;     // words of a workgroup's shapes at most

struct MergeLds {
  u64 t[kMergeWords], a[kMergeWords + 1], link[kMergeWords + 1], plane[2][2][kMergeWords + 1];
  uint32_t rank[kMergeWords], at[kMergeWords], word[kMergeWords], before[kMergeWords + 1], first[kMergeWords + 1], sum[kMergeWords / 64];
  uint16_t place[kGroupWords];             // of every word of the workgroup's shapes
};

// A workgroup takes the non-empty words of its shapes in batches, a lane per word; a word step further on a level axis
// is another lane's, found through `place`.  link = agree & equal extents on the axes inside the shape that are
// done (a pass clears `agree` of the later axes where the extents it made differ), and a chain has at most four boxes.
template <bool COST, int LV>
__device__ __forceinline__ void shape_merge(const RowGeo& g, const RowBufs& B, const RowWords& W, MergeLds& S, uint32_t group_words) {
  constexpr int kLevels = (int)kRowLevels;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  // its shapes lie far apart: the small ones, most of whose words have heads, are neighbours in the table
  const uint32_t block = spread_block();
  auto shape_of = [&](uint32_t local) { return (local >> g.lg_nw) * gridDim.x + block; };
  const size_t list = COST ? (size_t)B.tot[kRowsTotal] * g.en : 0;
  const size_t both = agree_stride(g, B.tot[kRowsTotal]);
  const u64* __restrict__ Tl = W.T + list;
  u64* __restrict__ left = COST ? W.Fk[1] : W.Fk[0];                   // (done with: the heads left, and in H's place
  u64* __restrict__ before = COST ? W.H[1] : W.H[0];                   //  the boxes of the shape before the word's)
  uint32_t* cnt = B.cnt + (COST ? g.n_shapes : 0u);
  for (uint32_t i = tid << g.lg_nw; i < group_words; i += 256u << g.lg_nw) if (shape_of(i) < g.n_shapes) cnt[shape_of(i)] = 0;
  if (tid == 0) {
    S.a[kNoWord] = S.link[kNoWord] = 0;
    for (int i = 0; i < 4; i++) S.plane[i >> 1][i & 1][kNoWord] = 0;
  }
  uint32_t c0 = 0, n_here = 0, mine_at = 0, chunk_n = 0, at_c = 0, rank_c = 0;
  u64 T_c = 0;
  bool have = false;
  for (;;) {
    // ---- fill the batch, 256 words (whole shapes) at a time ----
    while (c0 < group_words) {
      if (!have) {
        const uint32_t shape = shape_of(c0 + tid), w = (c0 + tid) & (g.nw - 1u);
        T_c = 0;
        if (shape < g.n_shapes && c0 + tid < group_words) {
          const uint32_t q = shape / g.en, n = shape - q * g.en, bm = q / g.ek, k = q - bm * g.ek, plane = (bm << g.lg_nw) + w;
          const uint32_t rows = B.rows[plane], first = B.first[plane];
          if (k < rows) {
            at_c = (first + k) * g.en + n;           // (fewer than 2^25 words)
            T_c = Tl[at_c];
            if (T_c) rank_c = W.rank[list + at_c].y;
          }
        }
        const u64 some = __ballot(T_c != 0);
        if (lane == 0) S.sum[wave] = (uint32_t)__popcll(some);
        __syncthreads();
        mine_at = below(some);
        chunk_n = 0;
        for (uint32_t x = 0; x < kMergeWords / 64; x++) { if (x < wave) mine_at += S.sum[x]; chunk_n += S.sum[x]; }
        chunk_n = (uint32_t)__builtin_amdgcn_readfirstlane((int)chunk_n);
        __syncthreads();
        have = true;
      }
      if (n_here + chunk_n > kMergeWords) break;
      const uint32_t slot = n_here + mine_at;
      if (T_c) { S.t[slot] = T_c; S.rank[slot] = rank_c; S.at[slot] = at_c; S.word[slot] = c0 + tid; }
      if (c0 + tid < kGroupWords) S.place[c0 + tid] = (uint16_t)(T_c ? slot : kNoWord);
      n_here += chunk_n;
      c0 += kMergeWords;
      have = false;
    }
    if (!n_here) return;
    __syncthreads();

    // ---- the lane's word and those next to it ----
    const uint32_t j = lane * (kMergeWords / 64) + wave;                // (few words: spread over the waves)
    const bool on = j < n_here;
    const u64 T = on ? S.t[j] : 0ull;
    const uint32_t local = on ? S.word[j] : 0u, w = local & (g.nw - 1u);
    const size_t at = list + (on ? S.at[j] : 0u);
    uint32_t next[kLevels], next2[kLevels], prev[kLevels];
    u64 lev[kLevels], var[LV ? LV : 1];
#pragma unroll
    for (int q = 0; q < kLevels; q++) lev[q] = on && (uint32_t)q < g.n_levels ? agree_level(g, W, both, q)[at] : 0ull;
#pragma unroll
    for (int b = 0; b < LV; b++) var[b] = on && field_at(g, b) ? agree_field(g, W, both, b)[at] : 0ull;
#pragma unroll
    for (int q = 0; q < kLevels; q++) {
      next[q] = next2[q] = prev[q] = kNoWord;
      const int sh = LV + 2 * q;
      if ((uint32_t)q >= g.n_levels || !on || sh < 5) continue;
      if (sh >= 6) {
        const uint32_t d = 1u << (sh >= 6 ? sh - 6 : 0), f = (w >> (sh >= 6 ? sh - 6 : 0)) & 3u;
        if (f < 3u) next[q] = S.place[local + d];
        if (f < 2u) next2[q] = S.place[local + 2u * d];
        if (f > 0u) prev[q] = S.place[local - d];
      } else if (!(w & 1u)) {
        next[q] = S.place[local + 1u];
      } else {
        prev[q] = S.place[local - 1u];
      }
    }

    // ---- the passes ----
    u64 A = T, ext[LV + 2 * kLevels];            // extent - 1 on an axis, at the axis's bits
#pragma unroll
    for (int i = 0; i < LV + 2 * kLevels; i++) ext[i] = 0;
#pragma unroll
    for (int q = 0; q < kLevels; q++) {
      if ((uint32_t)q >= g.n_levels) continue;
      const int sh = LV + 2 * q, in = sh < 5 ? 1 << sh : 0;
      u64 link, two, three, before;
      int any = 1;
      if (sh >= 5) {
        if (on) S.a[j] = A;
        __syncthreads();
        link = A & lev[q] & (sh >= 6 ? S.a[next[q]] : A >> 32 | S.a[next[q]] << 32);
        if (on) S.link[j] = link;
        any = __syncthreads_or(link != 0);
        if (sh >= 6) {
          two = link & S.link[next[q]];
          three = two & S.link[next2[q]];
          before = S.link[prev[q]];
        } else {
          const u64 up = S.link[next[q]];
          two = link & (link >> 32 | up << 32);
          three = two & up;
          before = link << 32 | S.link[prev[q]] >> 32;
        }
      } else {
        link = A & lev[q] & A >> in;
        two = link & link >> in;
        three = two & link >> (2 * in);
        before = link << in;
      }
      if (!any) continue;
      A &= ~before;
      const u64 e0 = (link & ~two) | three, e1 = two;
      ext[sh] = e0;
      ext[sh + 1] = e1;
      // the later axes: heads agree only with the same extent on this one
      const bool far = LV + 2 * ((int)g.n_levels - 1) >= 5 && q + 1 < (int)g.n_levels;
      if (far) {
        if (on) { S.plane[q & 1][0][j] = e0; S.plane[q & 1][1][j] = e1; }
        __syncthreads();
      }
#pragma unroll
      for (int p = q + 1; p < kLevels; p++) {
        if ((uint32_t)p >= g.n_levels) continue;
        const int s2 = LV + 2 * p, in2 = s2 < 5 ? 1 << s2 : 0;
        u64 o0, o1;
        if (s2 >= 6) { o0 = S.plane[q & 1][0][next[p]]; o1 = S.plane[q & 1][1][next[p]]; }
        else if (s2 == 5) { o0 = e0 >> 32 | S.plane[q & 1][0][next[p]] << 32; o1 = e1 >> 32 | S.plane[q & 1][1][next[p]] << 32; }
        else { o0 = e0 >> in2; o1 = e1 >> in2; }
        lev[p] &= ~((e0 ^ o0) | (e1 ^ o1));
      }
#pragma unroll
      for (int b = 0; b < LV; b++) var[b] &= ~((e0 ^ e0 >> (1 << b)) | (e1 ^ e1 >> (1 << b)));
    }
    // layout fields from the lowest up, then the dtype bits
#pragma unroll
    for (int half = 0; half < 2; half++)
#pragma unroll
      for (int b = 0; b < LV; b++) {
        if (!field_at(g, b) || (half == 0) != ((uint32_t)b >= g.ndt)) continue;
        const bool four = (g.var_two >> b) & 1u;
        const u64 link = A & var[b] & A >> (1 << b);
        const u64 two = four ? link & link >> (1 << b) : 0ull, three = four ? two & link >> (2 << b) : 0ull;
        A &= ~(link << (1 << b));
        const u64 e0 = (link & ~two) | three, e1 = two;
        ext[b] = e0;
        if (four && b + 1 < LV) ext[b + 1] = e1;
#pragma unroll
        for (int c = 0; c < LV; c++) var[c] &= c == b ? ~0ull : ~((e0 ^ e0 >> (1 << c)) | (e1 ^ e1 >> (1 << c)));
      }

    // ---- what is left: the heads, their extents inside the shape, boxes of the shape and before the word ----
    if (on) S.before[j] = (uint32_t)__popcll(A);
    __syncthreads();
    uint32_t own = tid < n_here ? S.before[tid] : 0u, incl = own;
    const bool starts = tid < n_here && (tid == 0 || (S.word[tid] >> g.lg_nw) != (S.word[tid - 1] >> g.lg_nw));
    const u64 start_mask = __ballot(starts);
    uint32_t shape_at = below(start_mask) + (starts ? 1u : 0u);        // shapes up to this one's
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(incl, d, 64);
      if ((int)lane >= d) incl += o;
    }
    if (lane == 63u) S.sum[wave] = incl | (uint32_t)__popcll(start_mask) << 16;      // (at most 16384 boxes, 256 shapes)
    __syncthreads();
    uint32_t excl = incl - own, total = 0, shapes = 0;
    for (uint32_t x = 0; x < kMergeWords / 64; x++) {
      const uint32_t s = S.sum[x];
      if (x < wave) { excl += s & 0xFFFFu; shape_at += s >> 16; }
      total += s & 0xFFFFu; shapes += s >> 16;
    }
    if (tid < n_here) S.before[tid] = excl;
    if (starts) S.first[shape_at - 1u] = tid;
    if (tid == 0) { S.before[n_here] = total; S.first[shapes] = n_here; }
    __syncthreads();
    if (tid < n_here) before[S.at[tid]] = excl - S.before[S.first[shape_at - 1u]];
    if (starts) cnt[shape_of(S.word[tid])] = S.before[S.first[shape_at]] - excl;
    if (on) {
      left[S.at[j]] = A;
      uint16_t* to = W.inner + S.rank[j];
      for (u64 todo = A; todo; todo &= todo - 1) {
        const uint32_t bit = (uint32_t)__builtin_ctzll(todo);
        uint32_t code = 0;
#pragma unroll
        for (int i = 0; i < LV + 2 * kLevels; i++) code |= ((uint32_t)(ext[i] >> bit) & 1u) << i;
        *to++ = (uint16_t)code;
      }
    }
    n_here = 0;
    __syncthreads();
  }
}

template <int LV>
__global__ __launch_bounds__(kMergeWords) void shape_merge_kernel(const RowGeo g, const RowBufs B, uint32_t group_words) {
  __shared__ MergeLds S;
  RowWords W;
  if (!row_words(g, B, W, true)) return;
  if (blockIdx.y == 0) shape_merge<true, LV>(g, B, W, S, group_words);
  else shape_merge<false, LV>(g, B, W, S, group_words);
}

template <int LV>
static void launch_inner(const RowGeo& g, const RowBufs& B, const uint64_t* cost, const uint16_t* arg, dim3 rows, hipStream_t st) {
  hipLaunchKernelGGL(row_inner_kernel<LV>, rows, dim3(256), 0, st, g, B, cost, arg);
  // words of a workgroup: as many as leave the chip 1024 workgroups and more
  const uint64_t words = (uint64_t)g.n_shapes << g.lg_nw;
  uint32_t group = g.nw;
  while (group < kGroupWords && words / (2 * group) >= 1024) group *= 2;
  hipLaunchKernelGGL(shape_merge_kernel<LV>, dim3((uint32_t)((words + group - 1) / group), 2), dim3(kMergeWords), 0, st, g, B, group);
}

// ---------------------------------------------------------------- the final lists
// Binary gcd (a 64-bit remainder is a long software routine here).
__device__ __forceinline__ int zeros_below(uint32_t x) { return __builtin_ctz(x); }
__device__ __forceinline__ int zeros_below(uint64_t x) { return __builtin_ctzll(x); }
template <class U>
__device__ __forceinline__ U reduce_by(U a, U b) {
  if (a == 0) return b;
  if (b == 0) return a;
  const int shift = zeros_below((U)(a | b));
  a >>= zeros_below(a);
  do {
    b >>= zeros_below(b);
    const U least = a < b ? a : b;
    b = a < b ? b - a : a - b;
    a = least;
  } while (b);
  return a << shift;
}

// The lane of a wave whose word has the wave's box i (excl: boxes of the lanes before).
__device__ __forceinline__ uint32_t lane_with(uint32_t excl, uint32_t i) {
  uint32_t at = 0;
#pragma unroll
  for (uint32_t d = 32; d > 0; d >>= 1) {
    const uint32_t there = (uint32_t)__shfl((int)excl, (int)(at + d), 64);
    at += there <= i ? d : 0u;
  }
  return at;
}

// A wave per row and list, its boxes a lane each.
__global__ __launch_bounds__(256) void row_emit_kernel(const RowGeo g, const RowBufs B, const uint64_t* __restrict__ cost,
                                                       const uint16_t* __restrict__ arg, const uint32_t* __restrict__ sizes) {
  RowWords W;
  if (!row_words(g, B, W, true)) return;
  const uint32_t lane = threadIdx.x & 63u, n_rows = B.tot[kRowsTotal], n0 = B.start[g.n_shapes], n_all = B.tot[kBoxesTotal];
  if (blockIdx.x == 0 && threadIdx.x == 0) B.tot[kBoxesFirst] = n0;
  const uint64_t lists = row_lists_at(g, B.tot);
  if (lists + row_list_bytes(n0) + row_list_bytes(n_all - n0) > B.room) return;
  const uint32_t parts = row_parts(g, n_rows);
  for (uint32_t ip = first_row(); ip < 2u * parts * n_rows; ip += gridDim.x * 4u) {
    const uint32_t part = ip % parts, i = ip / parts, l = i < n_rows ? 1u : 0u;
    const WaveRow r(B, l ? i : i - n_rows);
    const size_t at = (size_t)r.row * g.en + lane, at_l = (l ? (size_t)n_rows * g.en : 0) + at;
    u64 A = 0, N = 0;
    uint2 rank = make_uint2(0, 0);
    uint32_t out = 0;
    if (lane < g.en) {
      const u64 T = W.T[at_l], a = (l ? W.Fk[1] : W.Fk[0])[at];
      A = T ? a : 0ull;
    }
    if (A) {
      N = W.N[at_l];
      rank = W.rank[at_l];
      out = B.start[l * g.n_shapes + r.shape0 + lane] + (uint32_t)(l ? W.H[1] : W.H[0])[at] - (l ? n0 : 0u);
    }
    uint32_t excl = (uint32_t)__popcll(A);
    const uint32_t own = excl;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(excl, d, 64);
      if ((int)lane >= d) excl += o;
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)excl, 63);
    if (!total) continue;
    excl -= own;
    const uint64_t nf = l ? n_all - n0 : n0;
    char* p = B.dyn + lists + (l ? row_list_bytes(n0) : 0);
    uint32_t* fcell = (uint32_t*)p; p += up256(nf * 4);
    uint4* flen = (uint4*)p; p += up256(nf * 16);
    uint64_t* fv0 = (uint64_t*)p; p += up256(nf * 8);
    uint64_t* fv1 = (uint64_t*)p;
    const uint64_t vol = (uint64_t)axis_sizes(g, sizes, 0)[r.b] * axis_sizes(g, sizes, 1)[r.m] * axis_sizes(g, sizes, 2)[r.k];
    const uint32_t size_n = lane < g.en ? axis_sizes(g, sizes, 3)[lane] : 1u;
    for (uint32_t i0 = part * 64u; i0 < total; i0 += parts * 64u) {
      const uint32_t box = i0 + lane < total ? i0 + lane : total - 1u;
      const uint32_t n = lane_with(excl, box), nth = box - (uint32_t)__shfl((int)excl, (int)n, 64);
      const u64 a = (u64)(uint32_t)__shfl((int)(uint32_t)(A >> 32), (int)n, 64) << 32 | (uint32_t)__shfl((int)(uint32_t)A, (int)n, 64);
      const u64 nn = (u64)(uint32_t)__shfl((int)(uint32_t)(N >> 32), (int)n, 64) << 32 | (uint32_t)__shfl((int)(uint32_t)N, (int)n, 64);
      const uint32_t rank_n = (uint32_t)__shfl((int)rank.x, (int)n, 64), rank_t = (uint32_t)__shfl((int)rank.y, (int)n, 64);
      const uint32_t o = (uint32_t)__shfl((int)out, (int)n, 64) + nth, sn = (uint32_t)__shfl((int)size_n, (int)n, 64);
      if (i0 + lane >= total) continue;
      const uint32_t bit = nth_bit(a, nth), cell = (((r.shape0 + n) << g.lg_nw) + r.w) * 64u + bit;
      const uint64_t v = l ? cost[cell] : (uint64_t)arg[cell];
      const uint32_t code = W.inner[rank_t + nth];
      const uint32_t size_ext = (nn >> bit) & 1ull ? W.ext[rank_n + (uint32_t)__popcll(nn & ((1ull << bit) - 1ull))] : 0x01010101u;
      uint32_t L1 = 0x01010101u, L2 = L1, L3 = L1;
      auto put = [&](uint32_t axis, uint32_t x) {
        x <<= 8u * (axis & 3u);
        L1 += axis >> 2 == 1 ? x : 0u;
        L2 += axis >> 2 == 2 ? x : 0u;
        L3 += axis >> 2 == 3 ? x : 0u;
      };
#pragma unroll
      for (uint32_t q = 0; q < kRowLevels; q++)
        if (q < g.n_levels) put(g.level_axis - q, (code >> (g.lv + 2 * q)) & 3u);
#pragma unroll
      for (uint32_t b = 0; b < 6; b++)
        if (field_at(g, b)) put(g.var_axis[b], (code >> b) & ((g.var_two >> b) & 1u ? 3u : 1u));
      fcell[o] = cell;
      flen[o] = make_uint4(size_ext, L1, L2, L3);
      uint64_t v0 = v, v1 = 0;
      if (l && v != kInf) {
        const uint64_t all = vol * sn;
        if (((v | all) >> 32) == 0) {
          const uint32_t d = reduce_by((uint32_t)v, (uint32_t)all);
          v0 = (uint32_t)v / d; v1 = (uint32_t)all / d;
        } else {
          const uint64_t d = reduce_by(v, all);
          v0 = v / d; v1 = all / d;
        }
      }
      fv0[o] = v0;
      fv1[o] = v1;
    }
  }
}

// ---------------------------------------------------------------- prefix sums
// out[i] = the items before i, *total = all.  The number of items may be known to the GPU only: a fixed grid of
// workgroups, each with a stretch of whole tiles; first the stretches' sums, then every workgroup adds up those before its own.
constexpr uint32_t kSumGroups = 1024, kSumTile = 2048;

struct SumCounts {                   // n 32-bit numbers
  typedef uint32_t V;
  const uint32_t* p;
  uint32_t* to;
  uint32_t n;
  __device__ __forceinline__ uint32_t items() const { return n; }
  __device__ __forceinline__ void open() {}
  __device__ __forceinline__ V one(uint32_t i) const { return p[i]; }
  __device__ __forceinline__ void two(uint32_t i, V& x, V& y) const { const uint2 v = *(const uint2*)(p + i); x = v.x; y = v.y; }
  __device__ __forceinline__ void put(uint32_t i, V before, V) const { to[i] = before; }
};
struct SumHeads {                    // the bits of N and of T (in the high half) side by side
  typedef u64 V;
  RowGeo g;
  RowBufs B;
  const u64 *N, *T;
  u64* to;
  uint32_t n;
  __device__ __forceinline__ void open() {
    RowWords W;
    n = row_words(g, B, W) ? 2u * B.tot[kRowsTotal] * g.en : 0u;
    N = W.N; T = W.T; to = (u64*)W.rank;
  }
  __device__ __forceinline__ uint32_t items() const { return n; }
  __device__ __forceinline__ V one(uint32_t i) const { return (u64)(uint32_t)__popcll(T[i]) << 32 | (uint32_t)__popcll(N[i]); }
  __device__ __forceinline__ void two(uint32_t i, V& x, V& y) const {
    const ulonglong2 t = *(const ulonglong2*)(T + i), m = *(const ulonglong2*)(N + i);
    x = (u64)(uint32_t)__popcll(t.x) << 32 | (uint32_t)__popcll(m.x);
    y = (u64)(uint32_t)__popcll(t.y) << 32 | (uint32_t)__popcll(m.y);
  }
  __device__ __forceinline__ void put(uint32_t i, V before, V) const { to[i] = before; }
};

template <class V>
__device__ __forceinline__ V sum_over_group(V v, V* sh) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_down(v, d, 64);
  __syncthreads();
  if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}

// a pair of items per lane and row of 128, four rows per wave
template <class S>
__device__ __forceinline__ void sum_load(const S& s, uint32_t first, uint32_t n, typename S::V (&x)[4], typename S::V (&y)[4]) {
#pragma unroll
  for (uint32_t r = 0; r < 4; r++) {
    const uint32_t i = first + r * 128u;
    x[r] = y[r] = 0;
    if (i + 1 < n) s.two(i, x[r], y[r]);
    else if (i < n) x[r] = s.one(i);
  }
}

template <class S, bool APPLY>
__global__ __launch_bounds__(256) void sum_kernel(S s, typename S::V* __restrict__ sums, typename S::V* __restrict__ total) {
  typedef typename S::V V;
  __shared__ V sh[4];
  s.open();
  const uint32_t n = s.items(), tiles = (n + kSumTile - 1) / kSumTile, each = (tiles + gridDim.x - 1) / gridDim.x;
  const uint32_t t0 = blockIdx.x * each, t1 = t0 + each < tiles ? t0 + each : tiles;
  const uint32_t in_tile = (threadIdx.x >> 6) * 512u + (threadIdx.x & 63u) * 2u;
  V x[4], y[4], run = 0;
  if (!APPLY) {
    for (uint32_t t = t0; t < t1; t++) {
      sum_load(s, t * kSumTile + in_tile, n, x, y);
#pragma unroll
      for (int r = 0; r < 4; r++) run += x[r] + y[r];
    }
    run = sum_over_group(run, sh);
    if (threadIdx.x == 0) sums[blockIdx.x] = run;
    return;
  }
  if (t0 >= tiles && blockIdx.x != 0) return;
  for (uint32_t g = threadIdx.x; g < blockIdx.x; g += 256) run += sums[g];
  run = sum_over_group(run, sh);
  for (uint32_t t = t0; t < t1; t++) {
    sum_load(s, t * kSumTile + in_tile, n, x, y);
    V before[4], wave = 0;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      V incl = x[r] + y[r];
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const V o = __shfl_up(incl, d, 64);
        if ((int)(threadIdx.x & 63u) >= d) incl += o;
      }
      before[r] = wave + incl - x[r] - y[r];
      wave += __shfl(incl, 63, 64);
    }
    __syncthreads();
    if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = wave;
    __syncthreads();
    V base = run;
    for (uint32_t w = 0; w < (threadIdx.x >> 6); w++) base += sh[w];
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const uint32_t i = t * kSumTile + in_tile + r * 128u;
      if (i < n) s.put(i, base + before[r], x[r]);
      if (i + 1 < n) s.put(i + 1, base + before[r] + x[r], y[r]);
    }
    run += sh[0] + sh[1] + sh[2] + sh[3];
  }
  if (threadIdx.x == 0 && t1 == tiles) *total = run;
}

// bound: the most items there can be.
static uint32_t sum_groups(uint64_t bound) {
  const uint64_t tiles = (bound + kSumTile - 1) / kSumTile;
  return (uint32_t)(tiles < 1 ? 1 : tiles < kSumGroups ? tiles : kSumGroups);
}
template <class S>
static void launch_sum(const S& s, uint64_t bound, void* sums, uint32_t* total, hipStream_t st) {
  typedef typename S::V V;
  const uint32_t groups = sum_groups(bound);
  if (groups > 1) hipLaunchKernelGGL(HIP_KERNEL_NAME(sum_kernel<S, false>), dim3(groups), dim3(256), 0, st, s, (V*)sums, (V*)total);
  hipLaunchKernelGGL(HIP_KERNEL_NAME(sum_kernel<S, true>), dim3(groups), dim3(256), 0, st, s, (V*)sums, (V*)total);
}

// ---------------------------------------------------------------- launches
size_t rows_sum_bytes(const RowGeo& g) { return sum_groups(2 * ((uint64_t)g.n_shapes << g.lg_nw)) * 8; }      // (the words of both lists: the longest sum)
static_assert(sizeof(RowInfo) == kRowInfoBytes, "the caller makes room for it");

void launch_row_total(const RowGeo& g, const uint32_t* fitmap, uint32_t* total, hipStream_t st) {
  hipLaunchKernelGGL(row_total_kernel, dim3((g.n_planes + 255) / 256), dim3(256), 0, st, g, (const u64*)fitmap, total);
}

void launch_rows(const RowGeo& g, const RowBufs& B, const uint64_t* cost, const uint16_t* arg, const uint32_t* fitmap,
                 const uint32_t* sizes, hipStream_t st) {
  const u64* fit = (const u64*)fitmap;
  const dim3 wg(256);
  const uint64_t words = (uint64_t)g.n_shapes << g.lg_nw;
  hipLaunchKernelGGL(row_count_kernel, dim3((g.n_planes + 255) / 256), wg, 0, st, g, fit, B.rows);
  launch_sum(SumCounts{B.rows, B.first, g.n_planes}, g.n_planes, B.sum, B.tot + kRowsTotal, st);
  hipLaunchKernelGGL(row_info_kernel, dim3((uint32_t)(((uint64_t)g.n_planes * g.ek + 255) / 256)), wg, 0, st, g, B);
  const uint64_t most_rows = (uint64_t)g.n_planes * g.ek * 8;      // (row_parts)
  const dim3 rows((uint32_t)((most_rows + 3) / 4 < kRowGroups ? (most_rows + 3) / 4 : kRowGroups));
  hipLaunchKernelGGL(row_heads_kernel, rows, wg, 0, st, g, B, cost, arg, fit, sizes);
  if (g.eb > 1) hipLaunchKernelGGL(row_agree_kernel<4>, rows, wg, 0, st, g, B, cost, arg, sizes);
  else hipLaunchKernelGGL(row_agree_kernel<3>, rows, wg, 0, st, g, B, cost, arg, sizes);
  const dim3 per_plane((uint32_t)(((uint64_t)g.n_planes * g.en + 255) / 256), 2);
  // (a lane holds a step of a chain in same_behind)
  const bool long_k = g.ek > 64, long_m = g.em > 64;
  const dim3 per_chain((uint32_t)(((uint64_t)g.n_planes * g.en + 3) / 4), 2);
  if (g.em > 1) {
    if (long_k) hipLaunchKernelGGL(row_fold_long_k_kernel, per_chain, wg, 0, st, g, B, 0u);
    else hipLaunchKernelGGL(row_fold_m_kernel, per_plane, wg, 0, st, g, B);
  }
  if (g.eb > 1) {
    const uint64_t chains = (uint64_t)g.eb * g.nw * g.ek * g.en;
    if (long_k) hipLaunchKernelGGL(row_fold_long_k_kernel, per_chain, wg, 0, st, g, B, 1u);
    else hipLaunchKernelGGL(row_fold_b_k_kernel, per_plane, wg, 0, st, g, B);
    if (long_m) hipLaunchKernelGGL(row_fold_long_m_kernel, dim3((uint32_t)((chains + 3) / 4), 2), wg, 0, st, g, B);
    else hipLaunchKernelGGL(row_fold_b_m_kernel, dim3((uint32_t)((chains + 255) / 256), 2), wg, 0, st, g, B);
  }
  hipLaunchKernelGGL(row_left_kernel, dim3((uint32_t)((words + 255) / 256 < kRowGroups ? (words + 255) / 256 : kRowGroups)), wg, 0, st, g, B);
  launch_sum(SumHeads{g, B, nullptr, nullptr, nullptr, 0}, 2 * words, B.sum, B.tot + kLongTotal, st);
  hipLaunchKernelGGL(row_extent_kernel, rows, wg, 0, st, g, B);
  void (*const inner[7])(const RowGeo&, const RowBufs&, const uint64_t*, const uint16_t*, dim3, hipStream_t) = {
      launch_inner<0>, launch_inner<1>, launch_inner<2>, launch_inner<3>, launch_inner<4>, launch_inner<5>, launch_inner<6>};
  inner[g.lv](g, B, cost, arg, rows, st);
  launch_sum(SumCounts{B.cnt, B.start, 2 * g.n_shapes}, 2 * (uint64_t)g.n_shapes, B.sum, B.tot + kBoxesTotal, st);
  hipLaunchKernelGGL(row_emit_kernel, rows, wg, 0, st, g, B, cost, arg, sizes);
}

}  // namespace mrl
