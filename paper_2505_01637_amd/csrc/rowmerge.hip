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
// number stays on the GPU: nothing is read back before the merge has ended.
//
//   row_count_kernel   rows kept per plane (b, m, place), then a prefix sum
//   row_heads_kernel   a wave per row: H of both lists
//   row_agree_kernel   a wave per row: heads that agree, in value and run length, with the one before on k, m, b.  Along k
//                      that settles it: Fk
//   row_fold_*_kernel  Fm; Fb: chains along k (and m) compared
//   row_left_kernel    T, and N: its heads with an extent above 1 on some size axis (few, in the cost list); prefix sum over N
//   row_extent_kernel  the four extents of the heads in N
//   shape_merge_kernel the passes over the axes inside a shape, bitwise; the heads left are put on a pile
//   (prefix sum over the shapes' numbers of boxes)
//   row_emit_kernel    from the pile to their places in the two final lists
//
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

// ---------------------------------------------------------------- where things lie
// Word arrays of the kept rows, n_rows * en words each (N and its ranks: both lists' one after the other), the extents
// of N's heads, the pile.
struct RowWords {
  u64 *H[2], *Fk[2], *Fm[2], *Fb[2], *T[2], *N;
  uint32_t *rank, *ext;
  uint4* pile;               // cell, size extents, extents - 1 inside the shape, list
  uint32_t pile_room;
};

__host__ __device__ __forceinline__ uint64_t up256(uint64_t x) { return (x + 255) & ~255ull; }

__host__ __device__ __forceinline__ uint64_t row_word_bytes(const RowGeo& g, uint64_t n_rows) {
  const uint64_t one = up256(n_rows * g.en * 8), sets = 3 + (g.em > 1 ? 1 : 0) + (g.eb > 1 ? 1 : 0);
  return 2 * sets * one + up256(2 * n_rows * g.en * 8) + up256(2 * n_rows * g.en * 4);
}
__host__ __device__ __forceinline__ uint64_t row_list_bytes(uint64_t n) { return up256(n * 4) + up256(n * 16) + 2 * up256(n * 8); }
// Where the pile lies (behind the extents), and the lists.
__host__ __device__ __forceinline__ uint64_t row_pile_at(const RowGeo& g, const uint32_t* tot) { return row_word_bytes(g, tot[kRowsTotal]) + up256((uint64_t)tot[kLongTotal] * 4); }
__host__ __device__ __forceinline__ uint64_t row_lists_at(const RowGeo& g, const uint32_t* tot) { return row_pile_at(g, tot) + up256((uint64_t)tot[kBoxesTotal] * 16); }

bool rows_fit(const RowGeo& g, const uint32_t* tot, uint64_t room, uint64_t list_at[2], uint64_t* end) {
  // (a kernel that found no room left the totals behind it unset: in this order)
  if (row_word_bytes(g, tot[kRowsTotal]) > room || row_pile_at(g, tot) > room) return false;
  if (tot[kPiled] > (room - row_pile_at(g, tot)) / 16) return false;
  list_at[0] = row_lists_at(g, tot);
  list_at[1] = list_at[0] + row_list_bytes(tot[kBoxesFirst]);
  *end = list_at[1] + row_list_bytes(tot[kBoxesTotal] - tot[kBoxesFirst]);
  return *end <= room;
}

// false: the rows (or, with longs, the extents of N's heads) do not fit the scratch; every kernel then does nothing and
// the host finds out by the same sums.
__device__ __forceinline__ bool row_words(const RowGeo& g, const RowBufs& B, RowWords& W, bool longs = false) {
  const uint64_t n_rows = B.tot[kRowsTotal], one = up256(n_rows * g.en * 8);
  char* p = B.dyn;
  auto take = [&](uint64_t bytes) { char* at = p; p += bytes; return at; };
  W.H[0] = (u64*)take(one); W.H[1] = (u64*)take(one);
  W.Fk[0] = (u64*)take(one); W.Fk[1] = (u64*)take(one);
  W.T[0] = (u64*)take(one); W.T[1] = (u64*)take(one);
  const uint64_t for_m = g.em > 1 ? one : 0, for_b = g.eb > 1 ? one : 0;        // (not used where there is no such axis)
  W.Fm[0] = (u64*)take(for_m); W.Fm[1] = (u64*)take(for_m);
  W.Fb[0] = (u64*)take(for_b); W.Fb[1] = (u64*)take(for_b);
  W.N = (u64*)take(up256(2 * n_rows * g.en * 8));
  W.rank = (uint32_t*)take(up256(2 * n_rows * g.en * 4));
  W.ext = (uint32_t*)p; W.pile = nullptr; W.pile_room = 0;
  if ((uint64_t)(p - B.dyn) > B.room) return false;
  if (!longs) return true;
  const uint64_t at = row_pile_at(g, B.tot);
  if (at > B.room) return false;
  const uint64_t most = (B.room - at) / 16;
  W.pile = (uint4*)(B.dyn + at);
  W.pile_room = most < 0xFFFFFFFFull ? (uint32_t)most : 0xFFFFFFFFu;
  return true;
}

// Words of a row that is not kept: every cell (INF, NONE), one run along n, folded into the row before it on k.
__device__ __forceinline__ u64 gone_word(uint32_t n) { return n == 0 ? ~0ull : 0ull; }

// ---------------------------------------------------------------- rows
// Sizes ascend, and what fits a level at some size fits it at every smaller one (a layout that only some sizes have
// shares its word with the row-major one, which all have): a row has a fitting cell if its first step has one.
__global__ __launch_bounds__(256) void row_count_kernel(const RowGeo g, const u64* __restrict__ fit, uint32_t* __restrict__ rows, uint32_t* __restrict__ tot) {
  const uint32_t p = blockIdx.x * 256u + threadIdx.x;
  if (p == 0) tot[kPiled] = 0;
  if (p >= g.n_planes) return;
  const uint32_t w = p & (g.nw - 1u), bm = p >> g.lg_nw;
  const u64* f = fit + (((size_t)bm * g.ek * g.en) << g.lg_nw) + w;
  const size_t step = (size_t)g.en << g.lg_nw;
  uint32_t last = 0;
#pragma unroll 8
  for (uint32_t k = 0; k < g.ek; k++) last = f[k * step] ? k + 1u : last;
  rows[p] = last + 1u < g.ek ? last + 1u : g.ek;
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

// The row a wave has: workgroups of four rows of a plane.
struct WaveRow { uint32_t plane, k, row, w, bm, b, m, shape0; bool kept; };
__device__ __forceinline__ WaveRow wave_row(const RowGeo& g, const RowBufs& B) {
  WaveRow r;
  const uint32_t kc = (g.ek + 3u) / 4u;
  r.plane = blockIdx.x / kc;
  r.k = (blockIdx.x - r.plane * kc) * 4u + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  r.kept = r.k < B.rows[r.plane];
  r.row = B.first[r.plane] + r.k;
  r.w = r.plane & (g.nw - 1u); r.bm = r.plane >> g.lg_nw; r.b = r.bm / g.em; r.m = r.bm - r.b * g.em;
  r.shape0 = (r.bm * g.ek + r.k) * g.en;
  return r;
}

// Lanes on the cells of a word, walking n; what is decided is a ballot and stays in scalar registers (lane t of a
// vector register keeps step t's word for the store).
constexpr int kRowSteps = 8;              // steps whose reads are in flight together

__global__ __launch_bounds__(256) void row_heads_kernel(const RowGeo g, const RowBufs B, const uint64_t* __restrict__ cost,
                                                        const uint16_t* __restrict__ arg, const u64* __restrict__ fit,
                                                        const uint32_t* __restrict__ sizes) {
  const uint32_t lane = threadIdx.x & 63u;
  const WaveRow r = wave_row(g, B);
  RowWords W;
  if (!r.kept || !row_words(g, B, W)) return;
  const u64 words = lane < g.en ? fit[((size_t)(r.shape0 + lane) << g.lg_nw) + r.w] : 0ull;
  const uint32_t size_n = lane < g.en ? sizes[3 * kMaxSizes + lane] : 1u;
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

// Heads of row 0 (the wave's) and of a row before it whose runs are equally long: the next head above them, if any, is
// the same step in both rows.  Lane n has the words of step n; seen from the far end a step settles that where it has
// heads (both), passes it on where it has none (a prefix computation over the lanes).
__device__ __forceinline__ u64 same_runs(u64 h, u64 h1, uint32_t en) {
  const uint32_t lane = threadIdx.x & 63u;
  const u64 both = h & h1;
  u64 hit = lane < en ? both : ~0ull, pass = lane < en ? ~(h | h1) : 0ull;
  for (uint32_t d = 1; d < en; d <<= 1) {
    const uint32_t from = lane + d;
    u64 nh = (u64)(uint32_t)__shfl((int)(uint32_t)(hit >> 32), (int)from, 64) << 32 | (uint32_t)__shfl((int)(uint32_t)hit, (int)from, 64);
    u64 np = (u64)(uint32_t)__shfl((int)(uint32_t)(pass >> 32), (int)from, 64) << 32 | (uint32_t)__shfl((int)(uint32_t)pass, (int)from, 64);
    if (from >= 64u) { nh = ~0ull; np = 0; }
    hit |= pass & nh;
    pass &= np;
  }
  u64 above = (u64)(uint32_t)__shfl((int)(uint32_t)(hit >> 32), (int)(lane + 1u), 64) << 32 | (uint32_t)__shfl((int)(uint32_t)hit, (int)(lane + 1u), 64);
  u64 open = (u64)(uint32_t)__shfl((int)(uint32_t)(pass >> 32), (int)(lane + 1u), 64) << 32 | (uint32_t)__shfl((int)(uint32_t)pass, (int)(lane + 1u), 64);
  if (lane == 63u) { above = ~0ull; open = 0; }
  return both & (above | open);
}

constexpr int kAgreeSteps = 4;

template <int NX>
__global__ __launch_bounds__(256) void row_agree_kernel(const RowGeo g, const RowBufs B, const uint64_t* __restrict__ cost,
                                                        const uint16_t* __restrict__ arg, const uint32_t* __restrict__ sizes) {
  const uint32_t lane = threadIdx.x & 63u;
  const WaveRow r = wave_row(g, B);
  RowWords W;
  if (!r.kept || !row_words(g, B, W)) return;
  // rows 1 to 3: the ones before on k, m, b
  const uint32_t back[4] = {0, g.en, g.ek * g.en, g.em * g.ek * g.en};
  const uint32_t planes[4] = {r.plane, r.plane, r.plane - g.nw, r.plane - g.em * g.nw};
  const bool has[4] = {true, r.k > 0, r.m > 0, r.b > 0};
  const uint32_t sz[4] = {1u, sizes[2 * kMaxSizes + r.k], sizes[kMaxSizes + r.m], sizes[r.b]};
  const uint32_t sz1[4] = {1u, r.k ? sizes[2 * kMaxSizes + r.k - 1] : 1u, r.m ? sizes[kMaxSizes + r.m - 1] : 1u, r.b ? sizes[r.b - 1] : 1u};
  const size_t at = (size_t)r.row * g.en + lane;
  u64 h[2], cand[2][4];
#pragma unroll
  for (int l = 0; l < 2; l++) h[l] = lane < g.en ? W.H[l][at] : 0ull;
#pragma unroll
  for (int x = 1; x < NX; x++) {
    bool kept = has[x];
    size_t at1 = 0;
    if (x == 1) at1 = at - g.en;
    else if (kept) { kept = r.k < B.rows[planes[x]]; at1 = (size_t)(B.first[planes[x]] + r.k) * g.en + lane; }
#pragma unroll
    for (int l = 0; l < 2; l++) {
      cand[l][x] = 0;
      if (!has[x]) continue;
      const u64 h1 = lane < g.en ? (kept ? W.H[l][at1] : gone_word(lane)) : 0ull;
      cand[l][x] = same_runs(h[l], h1, g.en);
      if (lane >= g.en) cand[l][x] = 0;
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
  if (lane < g.en) {
#pragma unroll
    for (int l = 0; l < 2; l++) {
      W.Fk[l][at] = cand[l][1];
      if (g.em > 1) W.Fm[l][at] = cand[l][2];                     // (that agree: the kernels below decide)
      if (NX > 3) W.Fb[l][at] = cand[l][NX - 1];
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
    u64 f[kFoldRows], f1[kFoldRows], h[kFoldRows], h1[kFoldRows], agree[kFoldRows];
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      const int k = k0 - u;
      const size_t j = (size_t)(k > 0 ? k : 0) * g.en;
      const bool own = k >= 0 && (uint32_t)k < K, other = k >= 0 && (uint32_t)k < K1;
      f[u] = own ? Fk[at0 + j] : gone; f1[u] = other ? Fk[at1 + j] : gone;
      h[u] = own ? H[at0 + j] : gone; h1[u] = other ? H[at1 + j] : gone;
      agree[u] = own ? Fm[at0 + j] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      const int k = k0 - u;
      if (k >= 0 && (uint32_t)k < K) Fm[at0 + (size_t)k * g.en] = agree[u] & h[u] & ~f[u] & h1[u] & ~f1[u] & same;
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
      const int k = k0 - u;
      const size_t j = (size_t)(k > 0 ? k : 0) * g.en;
      const bool own = k >= 0 && (uint32_t)k < K, other = k >= 0 && (uint32_t)k < K1;
      f[u] = own ? Fk[at0 + j] : gone; f1[u] = other ? Fk[at1 + j] : gone;
      left[u] = own && other ? Fb[at0 + j] & H[at0 + j] & H[at1 + j] : 0ull;
      if (has_m && own && other) left[u] &= ~(Fm[at0 + j] | Fm[at1 + j]);
    }
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      const int k = k0 - u;
      if (k >= 0 && (uint32_t)k < K) Fb[at0 + (size_t)k * g.en] = left[u] & ~f[u] & ~f1[u] & same;
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
    for (int u = 0; u < kFoldRows; u++) {
      const int m = m0 - u;
      const uint32_t p = ((b * g.em + (uint32_t)(m > 0 ? m : 0)) << g.lg_nw) + w, p1 = p - g.em * g.nw;
      own[u] = m >= 0 && k < B.rows[p];
      const bool other = m >= 0 && k < B.rows[p1];
      at[u] = ((size_t)B.first[p] + (own[u] ? k : 0u)) * g.en + n;
      const size_t at1 = ((size_t)B.first[p1] + (other ? k : 0u)) * g.en + n;
      f[u] = g.em > 1 && own[u] ? Fm[at[u]] : 0ull; f1[u] = g.em > 1 && other ? Fm[at1] : 0ull;
      fold[u] = own[u] ? Fb[at[u]] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      if (own[u]) Fb[at[u]] = fold[u] & same;
      same = ~(f[u] ^ f1[u]) & (~f[u] | same);
    }
  }
}

// A lane per (plane, n), walking k: the heads left, and those of them that some row or step after theirs was folded into.
__global__ __launch_bounds__(256) void row_left_kernel(const RowGeo g, const RowBufs B) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x, l = blockIdx.y;
  const uint32_t p = i / g.en, n = i - p * g.en;
  if (p >= g.n_planes) return;
  RowWords W;
  if (!row_words(g, B, W)) return;
  const uint32_t bm = p >> g.lg_nw, b = bm / g.em, m = bm - b * g.em;
  const uint32_t K = B.rows[p], Km = m + 1u < g.em ? B.rows[p + g.nw] : 0u, Kb = b + 1u < g.eb ? B.rows[p + g.em * g.nw] : 0u;
  const size_t at0 = (size_t)B.first[p] * g.en + n, atm = Km ? (size_t)B.first[p + g.nw] * g.en + n : 0, atb = Kb ? (size_t)B.first[p + g.em * g.nw] * g.en + n : 0;
  const u64* __restrict__ H = l ? W.H[1] : W.H[0];
  const u64* __restrict__ Fk = l ? W.Fk[1] : W.Fk[0];
  const u64* __restrict__ Fm = l ? W.Fm[1] : W.Fm[0];
  const u64* __restrict__ Fb = l ? W.Fb[1] : W.Fb[0];
  u64* __restrict__ T = l ? W.T[1] : W.T[0];
  u64* __restrict__ N = W.N + (l ? (size_t)B.tot[kRowsTotal] * g.en : 0);
  u64 fk1 = K < g.ek ? gone_word(n) : 0ull;                    // Fk of the row after
  for (int k0 = (int)K - 1; k0 >= 0; k0 -= kFoldRows) {
    u64 f[kFoldRows], t[kFoldRows], more[kFoldRows];
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      const uint32_t k = k0 - u >= 0 ? (uint32_t)(k0 - u) : 0u;
      const size_t j = (size_t)k * g.en;
      f[u] = Fk[at0 + j];
      t[u] = H[at0 + j] & ~f[u];
      more[u] = n + 1u < g.en ? ~H[at0 + j + 1] : 0ull;
      if (g.em > 1) t[u] &= ~Fm[at0 + j];
      if (g.eb > 1) t[u] &= ~Fb[at0 + j];
      if (k < Km) more[u] |= Fm[atm + j];
      if (k < Kb) more[u] |= Fb[atb + j];
    }
#pragma unroll
    for (int u = 0; u < kFoldRows; u++) {
      if (k0 - u < 0) break;
      const size_t j = (size_t)(k0 - u) * g.en;
      T[at0 + j] = t[u];
      N[at0 + j] = t[u] & (more[u] | fk1);
      fk1 = f[u];
    }
  }
}

// ---------------------------------------------------------------- extents on the size axes
// A wave per row, the words with heads in N: the words further on along an axis are gathered, a lane each, and only the
// steps at which some chain ends are looked at.
__global__ __launch_bounds__(256) void row_extent_kernel(const RowGeo g, const RowBufs B) {
  const uint32_t lane = threadIdx.x & 63u, l = 1u - blockIdx.y;
  const WaveRow r = wave_row(g, B);
  RowWords W;
  if (!r.kept || !row_words(g, B, W, true)) return;
  const uint32_t plane = r.plane, k = r.k, row = r.row, b = r.b, m = r.m, K = B.rows[plane];
  const u64* Hl = l ? W.H[1] : W.H[0];
  const u64* Fk = l ? W.Fk[1] : W.Fk[0];
  const u64* Fm = l ? W.Fm[1] : W.Fm[0];
  const u64* Fb = l ? W.Fb[1] : W.Fb[0];
  const size_t at = (size_t)row * g.en + lane, at_t = (l ? (size_t)B.tot[kRowsTotal] * g.en : 0) + at;
  const bool mine = lane < g.en;
  const u64 t = mine ? W.N[at_t] : 0ull;
  u64 todo = __ballot(t != 0);
  if (!todo) return;
  const u64 h = mine ? Hl[at] : ~0ull;
  const uint32_t rank = mine ? W.rank[at_t] : 0u;
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
  const u64 long_m = mine && g.em > 1 ? t & word_m(1, lane) : 0ull;
  const u64 long_b = mine && g.eb > 1 ? t & word_b(1, lane) : 0ull;
  const u64 has_n = __ballot(long_n != 0), has_k = __ballot(long_k != 0), has_m = __ballot(long_m != 0), has_b = __ballot(long_b != 0);
  // cells of `cur` have extent 2 or more; word(c, n): the chain goes on to step c
  auto walk = [&](u64 cur, uint32_t n, uint32_t shift, uint32_t& e, auto&& word) {
    for (uint32_t c0 = 2; cur; c0 += 64) {
      const u64 on = word(c0 + lane, n);
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
    uint32_t e = 0x01010101u;                                   // b, m, k, n, a byte each
    if ((has_n >> n) & 1ull) {
      u64 cur = lane64(long_n, n);
      while (cur) {
        const u64 ends = __ballot(lane > n && ((h & cur) != 0 || lane >= g.en));
        const uint32_t c = ends ? (uint32_t)__builtin_ctzll(ends) : g.en;      // (64 steps: no lane is left to end the list)
        const u64 gone = c < g.en ? cur & lane64(h, c) : cur;
        if (in_mask(gone)) e += (c - n - 1u) << 24;
        cur &= ~gone;
      }
    }
    if ((has_k >> n) & 1ull) walk(lane64(long_k, n), n, 16, e, word_k);
    if ((has_m >> n) & 1ull) walk(lane64(long_m, n), n, 8, e, word_m);
    if ((has_b >> n) & 1ull) walk(lane64(long_b, n), n, 0, e, word_b);
    if (in_mask(tn)) W.ext[at_rank] = e;
  }
}

// ---------------------------------------------------------------- the axes inside a shape
constexpr uint32_t kMergeWords = 256;      // words of a batch, a lane each
constexpr uint32_t kNoWord = kMergeWords;  // LDS place of a word without heads
constexpr uint32_t kGroupWords = 2048;     // words of a workgroup's shapes at most

struct MergeLds {
  u64 t[kMergeWords + 1], n[kMergeWords + 1], a[kMergeWords + 1], link[kMergeWords + 1], plane[2][2][kMergeWords + 1];
  uint32_t rank[kMergeWords + 1], word[kMergeWords], before[kMergeWords + 1], first[kMergeWords + 1], sum[kMergeWords / 64], base;
  uint16_t place[kGroupWords];             // of every word of the workgroup's shapes
};

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

// A workgroup takes the non-empty words of its shapes in batches, a lane per word; a word step further on a level axis
// is another lane's, found through `place`.  First, which heads agree with the one a step further on an axis, in
// value and in size extents, for all axes at once (the lanes on the cells of one word after the other): nothing of
// that changes from pass to pass, as a head that is linked to has extent 1 on the axis.  Then the passes are word
// operations: link = agree & equal extents on the axes inside the shape that are done (a pass clears `agree` of the
// later axes where the extents it made differ), and a chain has at most four boxes.
// LV: bits of layouts and dtypes.
template <bool COST, int LV>
__device__ __forceinline__ void shape_merge(const RowGeo& g, const RowBufs& B, const RowWords& W, MergeLds& S, uint32_t group_words,
                                            const uint64_t* __restrict__ cost, const uint16_t* __restrict__ arg) {
  constexpr int kLevels = (int)kRowLevels;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t word0 = blockIdx.x * group_words, word_end = g.n_shapes << g.lg_nw;
  const size_t list = COST ? (size_t)B.tot[kRowsTotal] * g.en : 0;
  const u64* __restrict__ Tl = COST ? W.T[1] : W.T[0];
  uint32_t* cnt = B.cnt + (COST ? g.n_shapes : 0u);
  uint32_t* piled = B.piled + (COST ? g.n_shapes : 0u);
  for (uint32_t i = word0 + (tid << g.lg_nw); i < word0 + group_words && i < word_end; i += 256u << g.lg_nw) cnt[i >> g.lg_nw] = 0;
  if (tid == 0) {
    S.t[kNoWord] = S.n[kNoWord] = S.a[kNoWord] = S.link[kNoWord] = 0; S.rank[kNoWord] = 0;
    for (int i = 0; i < 4; i++) S.plane[i >> 1][i & 1][kNoWord] = 0;
  }
  uint32_t c0 = 0, n_here = 0, mine_at = 0, chunk_n = 0, rank_c = 0;
  u64 T_c = 0, N_c = 0;
  bool have = false;
  for (;;) {
    // ---- fill the batch, 256 words (whole shapes) at a time ----
    while (c0 < group_words) {
      if (!have) {
        const uint32_t i = word0 + c0 + tid, shape = i >> g.lg_nw, w = i & (g.nw - 1u);
        T_c = N_c = 0; rank_c = 0;
        if (i < word_end && c0 + tid < group_words) {
          const uint32_t q = shape / g.en, n = shape - q * g.en, bm = q / g.ek, k = q - bm * g.ek, plane = (bm << g.lg_nw) + w;
          if (k < B.rows[plane]) {
            const size_t at = (size_t)(B.first[plane] + k) * g.en + n;
            T_c = Tl[at];
            if (T_c) { N_c = W.N[list + at]; rank_c = W.rank[list + at]; }
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
      if (T_c) { S.t[slot] = T_c; S.n[slot] = N_c; S.rank[slot] = rank_c; S.word[slot] = c0 + tid; }
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
    const u64 T = on ? S.t[j] : 0ull, N = on ? S.n[j] : 0ull;
    const uint32_t rank = on ? S.rank[j] : 0u, local = on ? S.word[j] : 0u, w = local & (g.nw - 1u);
    uint32_t next[kLevels], next2[kLevels], prev[kLevels];
    u64 lev[kLevels], var[LV ? LV : 1];                                  // heads that agree with the one a step further
#pragma unroll
    for (int q = 0; q < kLevels; q++) {
      next[q] = next2[q] = prev[q] = kNoWord;
      lev[q] = 0;
      if ((uint32_t)q >= g.n_levels) continue;
      const int sh = LV + 2 * q;
      if (sh >= 6) {
        const uint32_t d = 1u << (sh >= 6 ? sh - 6 : 0), f = (w >> (sh >= 6 ? sh - 6 : 0)) & 3u;
        if (on) {
          if (f < 3u) next[q] = S.place[local + d];
          if (f < 2u) next2[q] = S.place[local + 2u * d];
          if (f > 0u) prev[q] = S.place[local - d];
        }
        lev[q] = T & S.t[next[q]] & ~(N ^ S.n[next[q]]);
      } else if (sh == 5) {
        if (on) {
          if (!(w & 1u)) next[q] = S.place[local + 1u];
          else prev[q] = S.place[local - 1u];
        }
        lev[q] = T & (T >> 32 | S.t[next[q]] << 32) & ~(N ^ (N >> 32 | S.n[next[q]] << 32)) & (w & 1u ? 0xFFFFFFFFull : ~0ull);
      } else {
        lev[q] = T & T >> (1 << (sh < 6 ? sh : 0)) & ~(N ^ N >> (1 << (sh < 6 ? sh : 0))) & not_last(sh, true);
      }
    }
#pragma unroll
    for (int b = 0; b < LV; b++) {
      var[b] = 0;
      if ((g.var_first >> b) & 1u) var[b] = T & T >> (1 << b) & ~(N ^ N >> (1 << b)) & not_last(b, (g.var_two >> b) & 1u);
    }

    // ---- values compared, the lanes on a word's cells ----
    u64 pairs = 0;
#pragma unroll
    for (int q = 0; q < kLevels; q++) pairs |= lev[q];
#pragma unroll
    for (int b = 0; b < LV; b++) pairs |= var[b];
    for (u64 todo = __ballot(pairs != 0); todo; todo &= todo - 1) {
      const uint32_t t = (uint32_t)__builtin_ctzll(todo);
      const size_t cell0 = (size_t)(word0 + (uint32_t)__builtin_amdgcn_readlane((int)local, (int)t)) * 64u;
      const uint64_t* c64 = cost + cell0;
      const uint16_t* a16 = arg + cell0;
      const u64 tw = lane64(T, t);
      uint64_t v = 0, v2[kLevels];
      u64 m[kLevels];
      if (in_mask(tw)) v = COST ? c64[lane] : (uint64_t)a16[lane];
#pragma unroll
      for (int q = 0; q < kLevels; q++) {
        m[q] = 0; v2[q] = 0;
        if ((uint32_t)q >= g.n_levels) continue;
        const int sh = LV + 2 * q;
        m[q] = lane64(lev[q], t);
        if (sh >= 5 && in_mask(m[q])) v2[q] = COST ? c64[(1u << sh) + lane] : (uint64_t)a16[(1u << sh) + lane];
      }
#pragma unroll
      for (int q = 0; q < kLevels; q++) {
        const int sh = LV + 2 * q;
        if ((uint32_t)q >= g.n_levels || !m[q]) continue;
        if (sh < 5) {
          v2[q] = step_above(sh, (uint32_t)v);
          if (COST) v2[q] |= (uint64_t)step_above(sh, (uint32_t)(v >> 32)) << 32;
        }
        put_lane64(lev[q], m[q] & __ballot(v == v2[q]), t);
      }
#pragma unroll
      for (int b = 0; b < LV; b++) {
        const u64 mb = lane64(var[b], t);
        if (!mb) continue;
        uint64_t vb = step_above(b, (uint32_t)v);
        if (COST) vb |= (uint64_t)step_above(b, (uint32_t)(v >> 32)) << 32;
        put_lane64(var[b], mb & __ballot(v == vb), t);
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
        if (sh >= 6) {
          const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)next[q], (int)t);
          const uint32_t at = S.rank[o] + below(S.n[o]);
          if (in_mask(m & nw)) e2 = W.ext[at];
        } else {
          e2 = (uint32_t)__shfl((int)e, (int)(lane + (1u << (sh < 6 ? sh : 0))), 64);
          if (sh == 5) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)next[q], (int)t);
            const uint32_t at = S.rank[o] + __popc((uint32_t)S.n[o] & ((1u << (lane & 31u)) - 1u));
            if (lane >= 32u && in_mask(m & nw)) e2 = W.ext[at];
          }
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
        if (!((g.var_first >> b) & 1u) || (half == 0) != ((uint32_t)b >= g.ndt)) continue;
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

    // ---- what is left goes on the pile, shape by shape ----
    if (on) S.before[j] = (uint32_t)__popcll(A);
    __syncthreads();
    uint32_t own = tid < n_here ? S.before[tid] : 0u, incl = own;
    const bool starts = tid < n_here && (tid == 0 || (S.word[tid] >> g.lg_nw) != (S.word[tid - 1] >> g.lg_nw));
    const u64 start_mask = __ballot(starts);
    uint32_t first_at = below(start_mask);
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
      if (x < wave) { excl += s & 0xFFFFu; first_at += s >> 16; }
      total += s & 0xFFFFu; shapes += s >> 16;
    }
    if (tid < n_here) S.before[tid] = excl;
    if (starts) S.first[first_at] = tid;
    if (tid == 0) {
      S.before[n_here] = total;
      S.first[shapes] = n_here;
      S.base = total ? atomicAdd(&B.tot[kPiled], total) : 0u;
    }
    __syncthreads();
    const uint32_t base = S.base;
    if (starts) {
      const uint32_t shape = (word0 + S.word[tid]) >> g.lg_nw;
      cnt[shape] = S.before[S.first[first_at + 1]] - excl;
      piled[shape] = base + excl;
    }
    if (base + total >= base && base + total <= W.pile_room) {
      uint32_t o = base + (on ? S.before[j] : 0u);
      const uint32_t cell0 = (word0 + local) * 64u;
      for (u64 left = A; left; left &= left - 1) {
        const uint32_t bit = (uint32_t)__builtin_ctzll(left);
        uint32_t code = 0;
#pragma unroll
        for (int i = 0; i < LV + 2 * kLevels; i++) code |= ((uint32_t)(ext[i] >> bit) & 1u) << i;
        const u64 under = (1ull << bit) - 1ull;
        const uint32_t e = (N >> bit) & 1ull ? W.ext[rank + (uint32_t)__popcll(N & under)] : 0x01010101u;
        W.pile[o++] = make_uint4(cell0 + bit, e, code, COST ? 1u : 0u);
      }
    }
    n_here = 0;
    __syncthreads();
  }
}

template <int LV>
__global__ __launch_bounds__(kMergeWords) void shape_merge_kernel(const RowGeo g, const RowBufs B, uint32_t group_words, const uint64_t* __restrict__ cost,
                                                                  const uint16_t* __restrict__ arg) {
  __shared__ MergeLds S;
  RowWords W;
  if (!row_words(g, B, W, true)) return;
  if (blockIdx.y == 0) shape_merge<true, LV>(g, B, W, S, group_words, cost, arg);
  else shape_merge<false, LV>(g, B, W, S, group_words, cost, arg);
}

static void launch_shape_merge(const RowGeo& g, const RowBufs& B, const uint64_t* cost, const uint16_t* arg, hipStream_t st) {
  // words of a workgroup: as many as leave the chip 2048 workgroups
  const uint64_t words = (uint64_t)g.n_shapes << g.lg_nw;
  uint32_t group = g.nw;
  while (group < kGroupWords && words / (2 * group) >= 2048) group *= 2;
  const dim3 grid((uint32_t)((words + group - 1) / group), 2);
  void (*const kernels[7])(const RowGeo, const RowBufs, uint32_t, const uint64_t*, const uint16_t*) = {
      shape_merge_kernel<0>, shape_merge_kernel<1>, shape_merge_kernel<2>, shape_merge_kernel<3>, shape_merge_kernel<4>, shape_merge_kernel<5>, shape_merge_kernel<6>};
  hipLaunchKernelGGL(kernels[g.lv], grid, dim3(kMergeWords), 0, st, g, B, group, cost, arg);
}

// ---------------------------------------------------------------- the final lists
// Binary gcd (a 64-bit remainder is a long software routine here).
__device__ __forceinline__ uint64_t reduce_by(uint64_t a, uint64_t b) {
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

// A lane per box on the pile: its place is its shape's first place plus how far it lies behind the shape's first on the pile.
constexpr uint32_t kEmitGroups = 4096;

__global__ __launch_bounds__(256) void row_emit_kernel(const RowGeo g, const RowBufs B, const uint64_t* __restrict__ cost,
                                                       const uint16_t* __restrict__ arg, const uint32_t* __restrict__ sizes) {
  RowWords W;
  if (!row_words(g, B, W, true) || B.tot[kPiled] > W.pile_room) return;
  const uint32_t n0 = B.start[g.n_shapes], n_all = B.tot[kBoxesTotal];
  if (blockIdx.x == 0 && threadIdx.x == 0) B.tot[kBoxesFirst] = n0;
  const uint64_t at = row_lists_at(g, B.tot);
  if (at + row_list_bytes(n0) + row_list_bytes(n_all - n0) > B.room) return;
  for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n_all; i += gridDim.x * 256u) {
    const uint4 box = W.pile[i];
    const uint32_t l = box.w, cell = box.x, code = box.z, shape = cell / g.G;
    const uint32_t o = B.start[l * g.n_shapes + shape] + (i - B.piled[l * g.n_shapes + shape]) - (l ? n0 : 0u);
    const uint64_t nf = l ? n_all - n0 : n0;
    char* p = B.dyn + at + (l ? row_list_bytes(n0) : 0);
    uint32_t* fcell = (uint32_t*)p; p += up256(nf * 4);
    uint4* flen = (uint4*)p; p += up256(nf * 16);
    uint64_t* fv0 = (uint64_t*)p; p += up256(nf * 8);
    uint64_t* fv1 = (uint64_t*)p;
    const uint64_t v = l ? cost[cell] : (uint64_t)arg[cell];
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
      if ((g.var_first >> b) & 1u) put(g.var_axis[b], (code >> b) & ((g.var_two >> b) & 1u ? 3u : 1u));
    fcell[o] = cell;
    flen[o] = make_uint4(box.y, L1, L2, L3);
    uint64_t v0 = v, v1 = 0;
    if (l && v != kInf) {
      uint32_t q = shape;
      uint64_t vol = 1;
      vol *= sizes[3 * kMaxSizes + q % g.en]; q /= g.en;
      vol *= sizes[2 * kMaxSizes + q % g.ek]; q /= g.ek;
      vol *= sizes[kMaxSizes + q % g.em]; q /= g.em;
      vol *= sizes[q];
      const uint64_t d = reduce_by(v, vol);
      v0 = v / d; v1 = vol / d;
    }
    fv0[o] = v0;
    fv1[o] = v1;
  }
}

// ---------------------------------------------------------------- prefix sums
// out[i] = the items before i, *total = all.  The number of items may be known to the GPU only: a fixed grid of
// workgroups, each with a stretch of whole tiles; first the stretches' sums, then every workgroup adds up those before its own.
constexpr uint32_t kSumGroups = 1024, kSumTile = 2048;

struct SumCounts {                   // n 32-bit numbers
  const uint32_t* p;
  uint32_t* to;
  uint32_t* sum;
  uint32_t n;
  __device__ __forceinline__ bool open(const uint32_t*& in, const u64*&, uint32_t*& out, uint32_t& count) const { in = p; out = to; count = n; return true; }
};
struct SumLong {                     // the bits of N
  RowGeo g;
  RowBufs B;
  uint32_t* sum;
  __device__ __forceinline__ bool open(const uint32_t*&, const u64*& in, uint32_t*& out, uint32_t& count) const {
    RowWords W;
    const bool fits = row_words(g, B, W);
    in = W.N; out = W.rank; count = fits ? 2u * B.tot[kRowsTotal] * g.en : 0u;
    return false;
  }
};

__device__ __forceinline__ uint32_t sum_over_group(uint32_t v, uint32_t* sh) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_down(v, d, 64);
  __syncthreads();
  if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}

// a pair of items per lane and row of 128, four rows per wave
template <class S>
__device__ __forceinline__ void sum_load(bool counts, const uint32_t* p, const u64* words, uint32_t first, uint32_t n, uint32_t (&x)[4], uint32_t (&y)[4]) {
#pragma unroll
  for (uint32_t r = 0; r < 4; r++) {
    const uint32_t i = first + r * 128u;
    x[r] = y[r] = 0;
    if (counts) {
      if (i + 1 < n) { const uint2 v = *(const uint2*)(p + i); x[r] = v.x; y[r] = v.y; }
      else if (i < n) x[r] = p[i];
    } else {
      if (i + 1 < n) { const ulonglong2 v = *(const ulonglong2*)(words + i); x[r] = (uint32_t)__popcll(v.x); y[r] = (uint32_t)__popcll(v.y); }
      else if (i < n) x[r] = (uint32_t)__popcll(words[i]);
    }
  }
}

template <class S, bool APPLY>
__global__ __launch_bounds__(256) void sum_kernel(const S s, uint32_t* __restrict__ total) {
  __shared__ uint32_t sh[4];
  const uint32_t* p = nullptr;
  const u64* words = nullptr;
  uint32_t* out = nullptr;
  uint32_t n = 0;
  const bool counts = s.open(p, words, out, n);
  const uint32_t tiles = (n + kSumTile - 1) / kSumTile, each = (tiles + gridDim.x - 1) / gridDim.x;
  const uint32_t t0 = blockIdx.x * each, t1 = t0 + each < tiles ? t0 + each : tiles;
  const uint32_t in_tile = (threadIdx.x >> 6) * 512u + (threadIdx.x & 63u) * 2u;
  uint32_t x[4], y[4], run = 0;
  if (!APPLY) {
    for (uint32_t t = t0; t < t1; t++) {
      sum_load<S>(counts, p, words, t * kSumTile + in_tile, n, x, y);
#pragma unroll
      for (int r = 0; r < 4; r++) run += x[r] + y[r];
    }
    run = sum_over_group(run, sh);
    if (threadIdx.x == 0) s.sum[blockIdx.x] = run;
    return;
  }
  if (t0 >= tiles && blockIdx.x != 0) return;
  for (uint32_t g = threadIdx.x; g < blockIdx.x; g += 256) run += s.sum[g];
  run = sum_over_group(run, sh);
  for (uint32_t t = t0; t < t1; t++) {
    sum_load<S>(counts, p, words, t * kSumTile + in_tile, n, x, y);
    uint32_t before[4], wave = 0;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      uint32_t incl = x[r] + y[r];
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, 64);
        if ((int)(threadIdx.x & 63u) >= d) incl += o;
      }
      before[r] = wave + incl - x[r] - y[r];
      wave += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
    __syncthreads();
    if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = wave;
    __syncthreads();
    uint32_t base = run;
    for (uint32_t w = 0; w < (threadIdx.x >> 6); w++) base += sh[w];
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const uint32_t i = t * kSumTile + in_tile + r * 128u, at = base + before[r];
      if (i + 1 < n) *(uint2*)(out + i) = make_uint2(at, at + x[r]);
      else if (i < n) out[i] = at;
    }
    run += sh[0] + sh[1] + sh[2] + sh[3];
  }
  if (threadIdx.x == 0 && (t1 == tiles)) *total = run;
}

// bound: the most items there can be.
template <class S>
static void launch_sum(const S& s, uint64_t bound, uint32_t* total, hipStream_t st) {
  const uint64_t tiles = (bound + kSumTile - 1) / kSumTile;
  const uint32_t groups = (uint32_t)(tiles < 1 ? 1 : tiles < kSumGroups ? tiles : kSumGroups);
  if (groups > 1) hipLaunchKernelGGL(HIP_KERNEL_NAME(sum_kernel<S, false>), dim3(groups), dim3(256), 0, st, s, total);
  hipLaunchKernelGGL(HIP_KERNEL_NAME(sum_kernel<S, true>), dim3(groups), dim3(256), 0, st, s, total);
}

// ---------------------------------------------------------------- launches
size_t rows_sum_bytes() { return kSumGroups * 4; }

void launch_rows(const RowGeo& g, const RowBufs& B, const uint64_t* cost, const uint16_t* arg, const uint32_t* fitmap,
                 const uint32_t* sizes, hipStream_t st) {
  const u64* fit = (const u64*)fitmap;
  const dim3 wg(256);
  const uint64_t words = (uint64_t)g.n_shapes << g.lg_nw;
  hipLaunchKernelGGL(row_count_kernel, dim3((g.n_planes + 255) / 256), wg, 0, st, g, fit, B.rows, B.tot);
  launch_sum(SumCounts{B.rows, B.first, B.sum, g.n_planes}, g.n_planes, B.tot + kRowsTotal, st);
  const uint32_t row_blocks = g.n_planes * ((g.ek + 3) / 4);
  hipLaunchKernelGGL(row_heads_kernel, dim3(row_blocks), wg, 0, st, g, B, cost, arg, fit, sizes);
  if (g.eb > 1) hipLaunchKernelGGL(row_agree_kernel<4>, dim3(row_blocks), wg, 0, st, g, B, cost, arg, sizes);
  else hipLaunchKernelGGL(row_agree_kernel<3>, dim3(row_blocks), wg, 0, st, g, B, cost, arg, sizes);
  const dim3 per_plane((uint32_t)(((uint64_t)g.n_planes * g.en + 255) / 256), 2);
  if (g.em > 1) hipLaunchKernelGGL(row_fold_m_kernel, per_plane, wg, 0, st, g, B);
  if (g.eb > 1) {
    hipLaunchKernelGGL(row_fold_b_k_kernel, per_plane, wg, 0, st, g, B);
    hipLaunchKernelGGL(row_fold_b_m_kernel, dim3((uint32_t)(((uint64_t)g.eb * g.nw * g.ek * g.en + 255) / 256), 2), wg, 0, st, g, B);
  }
  hipLaunchKernelGGL(row_left_kernel, per_plane, wg, 0, st, g, B);
  launch_sum(SumLong{g, B, B.sum}, 2 * words, B.tot + kLongTotal, st);
  hipLaunchKernelGGL(row_extent_kernel, dim3(row_blocks, 2), wg, 0, st, g, B);
  launch_shape_merge(g, B, cost, arg, st);
  launch_sum(SumCounts{B.cnt, B.start, B.sum, 2 * g.n_shapes}, 2 * (uint64_t)g.n_shapes, B.tot + kBoxesTotal, st);
  hipLaunchKernelGGL(row_emit_kernel, dim3(kEmitGroups), wg, 0, st, g, B, cost, arg, sizes);
}

}  // namespace mrl
