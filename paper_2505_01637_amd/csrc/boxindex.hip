// Point lookups in a final box list (Section 4.1: the table is kept as boxes and a lookup finds
// the box that holds a Spec's coordinate).
//
// The boxes of a list are disjoint, cover the lattice and are sorted by their low corner in
// row-major order.  Over that order sits a packed hierarchy of bounding boxes with fan-out 8
// (level 0: the boxes themselves; a node of level l+1 bounds 8 consecutive nodes of level l),
// i.e. an R-tree bulk-loaded in the list's own order.  A lookup walks it depth first and descends
// only into nodes whose bounds contain the point; exactly one box of level 0 does.
#include <hip/hip_runtime.h>

#include "compress.h"

namespace mrl {

namespace {

// Bit 7 of every byte: whether x >= y there (the low seven bits by a subtraction that borrows from
// no neighbour, the top bits by themselves).
__device__ __forceinline__ uint32_t bytes_ge(uint32_t x, uint32_t y) {
  const uint32_t t = (x | 0x80808080u) - (y & 0x7F7F7F7Fu), d = x ^ y;
  return (d & x) | (~d & t);
}

__device__ __forceinline__ bool contains(const uint4& lo, const uint4& hi, const uint4& p) {
  const uint32_t in = bytes_ge(p.x, lo.x) & bytes_ge(p.y, lo.y) & bytes_ge(p.z, lo.z) & bytes_ge(p.w, lo.w) &
                      bytes_ge(hi.x, p.x) & bytes_ge(hi.y, p.y) & bytes_ge(hi.z, p.z) & bytes_ge(hi.w, p.w);
  return (in & 0x80808080u) == 0x80808080u;
}

// Level 0: corners of each box from its low cell and its run lengths.  Axes beyond ndim get
// lo = hi = 0, which every point (padded with zeros) satisfies.
__global__ __launch_bounds__(256) void box_bounds_kernel(Geo g, uint32_t n, const uint32_t* __restrict__ fcell,
                                                         const uint8_t* __restrict__ flen, BoxBounds* __restrict__ out) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  BoxBounds b;
  uint32_t x = fcell[i];
#pragma unroll
  for (uint32_t a = 0; a < 16; a++) {
    uint32_t lo = 0, len = 1;
    if (a < g.ndim) {
      lo = x / g.stride[a];
      x -= lo * g.stride[a];
      len = flen[(size_t)i * 16 + a];
    }
    b.lo[a] = (uint8_t)lo;
    b.hi[a] = (uint8_t)(lo + len - 1);
  }
  out[i] = b;
}

__global__ __launch_bounds__(256) void group_bounds_kernel(const BoxBounds* __restrict__ in, uint32_t n_in,
                                                           BoxBounds* __restrict__ out, uint32_t n_out) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n_out) return;
  BoxBounds r;
#pragma unroll
  for (int a = 0; a < 16; a++) { r.lo[a] = 255; r.hi[a] = 0; }
  const uint32_t first = i * kIndexFan;
  const uint32_t last = min(first + kIndexFan, n_in);
  for (uint32_t c = first; c < last; c++) {
    const BoxBounds b = in[c];
#pragma unroll
    for (int a = 0; a < 16; a++) {
      r.lo[a] = min(r.lo[a], b.lo[a]);
      r.hi[a] = max(r.hi[a], b.hi[a]);
    }
  }
  out[i] = r;
}

// Eight lanes per point, a lane per node of a group of siblings: one test of a group is one read of
// 256 bytes by the eight of them and a ballot.  (A lane per point tested the nodes one after the
// other, each test waiting for a read of its own: 65,536 points in lists of 21,556 and 398,016 boxes
// took 1.87 ms, with eight lanes 0.28 ms.)
// The boxes are sorted by low corner in row-major order and the box that holds a point starts at or
// before the point in that order.  So first the last box that starts there is looked for, from the
// top of the hierarchy, eight starts at a time; then the walk runs backwards from it, as the box
// wanted is usually a few boxes away: the siblings before it, the siblings before its parent with
// what is below them, and so on.  Every group is tested at most once, so the walk ends.
// blockIdx.y: the list, decisions or costs.  A point that lies in no box (the list is then not a
// partition) is marked in miss[list] for the host to report.
constexpr uint32_t kLookupPoints = 256 / kIndexFan;       // per workgroup

struct LookupLists { LookupList list[2]; };

__global__ __launch_bounds__(256) void lookup_kernel(Geo g, LookupLists lists, const uint4* __restrict__ points,
                                                     const uint64_t* __restrict__ vols, uint32_t n_points,
                                                     uint64_t* __restrict__ cost_out, uint16_t* __restrict__ arg_out,
                                                     uint8_t* __restrict__ miss) {
  const bool is_cost = blockIdx.y != 0;
  const LookupList& T = lists.list[blockIdx.y];
  __shared__ uint32_t count[kIndexMaxLevels], off[kIndexMaxLevels];
  if (threadIdx.x < kIndexMaxLevels) {
    count[threadIdx.x] = T.L.count[threadIdx.x];
    off[threadIdx.x] = T.L.off[threadIdx.x];
  }
  __syncthreads();
  const BoxBounds* __restrict__ nodes = T.nodes;
  const uint32_t* __restrict__ fcell = T.fcell;
  const uint32_t n_levels = T.L.n_levels;
  const uint32_t q = blockIdx.x * kLookupPoints + threadIdx.x / kIndexFan, sub = threadIdx.x % kIndexFan;
  const uint32_t shift = threadIdx.x & 63u & ~(kIndexFan - 1u);       // the eight lanes' place in a ballot
  if (q >= n_points) return;                                          // all eight of them
  const uint4 p = points[q];
  uint32_t cell = 0;
#pragma unroll
  for (uint32_t a = 0; a < 16; a++) {
    const uint32_t w = a < 4 ? p.x : a < 8 ? p.y : a < 12 ? p.z : p.w;
    if (a < g.ndim) cell += ((w >> (8 * (a & 3u))) & 0xFFu) * g.stride[a];
  }
  // pos: the last box whose first cell is <= the point's (box 0 starts at cell 0)
  uint32_t pos = 0;
  for (uint32_t l = n_levels; l-- > 0;) {
    const uint32_t i = pos * kIndexFan + sub;
    const bool before = i < count[l] && fcell[(size_t)i << (3 * l)] <= cell;
    const uint32_t m = (uint32_t)(__ballot(before) >> shift) & 0xFFu;
    pos = pos * kIndexFan + (m ? (uint32_t)__popc(m) - 1u : 0u);
  }
  // which of the nodes of a group hold the point
  auto test = [&](uint32_t l, uint32_t group) -> uint32_t {
    const uint32_t i = group * kIndexFan + sub;
    bool in = false;
    if (i < count[l]) {
      const uint4* b = reinterpret_cast<const uint4*>(nodes + off[l] + i);
      in = contains(b[0], b[1], p);
    }
    return (uint32_t)(__ballot(in) >> shift) & 0xFFu;
  };
  uint32_t found = 0xFFFFFFFFu;
  for (uint32_t up = 0; up < n_levels && found == 0xFFFFFFFFu; up++) {
    const uint32_t at = pos >> (3 * up);
    uint32_t l = up, group = at >> 3;
    // the siblings before the node that pos is in (among the boxes themselves, pos as well)
    uint32_t m = test(l, group) & ((up == 0 ? 2u : 1u) << (at & 7u)) - 1u;
    // what is left to try on the levels above l, a byte each, the nearest lowest
    uint64_t left = 0;
    uint32_t left_hi = 0;
    while (true) {
      while (m == 0 && l < up) {
        l++;
        group >>= 3;
        m = (uint32_t)left & 0xFFu;
        left = left >> 8 | (uint64_t)left_hi << 56;
        left_hi >>= 8;
      }
      if (m == 0) break;
      const uint32_t top = 31u - (uint32_t)__clz((int)m);
      group = group * kIndexFan + top;
      if (l == 0) { found = group; break; }
      left_hi = left_hi << 8 | (uint32_t)(left >> 56);
      left = left << 8 | (m & ~(1u << top));
      l--;
      m = test(l, group);
    }
  }
  if (sub != 0) return;
  const bool hit = found != 0xFFFFFFFFu;
  miss[(is_cost ? n_points : 0u) + q] = hit ? 0 : 1;
  if (!is_cost) {
    arg_out[q] = hit ? (uint16_t)T.fv0[found] : 0;
  } else {
    // the box's cost per volume is the reduced fraction v0 / v1 and the point's cost is v0 * volume / v1,
    // a whole number: v1, which shares no factor with v0, divides the volume.  v1 = 0: no implementation.
    const uint64_t v0 = hit ? T.fv0[found] : 0, v1 = hit ? T.fv1[found] : 1;
    cost_out[q] = v1 == 0 ? kInf : v0 * (vols[q] / v1);
  }
}

}  // namespace

IndexLevels index_levels(uint32_t n_boxes) {
  IndexLevels L;
  L.n_levels = 0;
  L.total = 0;
  uint32_t n = n_boxes;
  while (true) {
    L.count[L.n_levels] = n;
    L.off[L.n_levels] = L.total;
    L.total += n;
    L.n_levels++;
    if (n <= kIndexFan || L.n_levels == kIndexMaxLevels) break;
    n = (n + kIndexFan - 1) / kIndexFan;
  }
  return L;
}

void launch_build_index(const Geo& g, const IndexLevels& L, const uint32_t* fcell, const void* flen, BoxBounds* nodes,
                        hipStream_t st) {
  const uint32_t n = L.count[0];
  if (!n) return;
  hipLaunchKernelGGL(box_bounds_kernel, dim3((n + 255) / 256), dim3(256), 0, st, g, n, fcell, (const uint8_t*)flen, nodes);
  for (uint32_t l = 1; l < L.n_levels; l++)
    hipLaunchKernelGGL(group_bounds_kernel, dim3((L.count[l] + 255) / 256), dim3(256), 0, st, nodes + L.off[l - 1],
                       L.count[l - 1], nodes + L.off[l], L.count[l]);
}

hipError_t launch_lookup(const Geo& g, const LookupList lists[2], const void* points, const uint64_t* vols, uint32_t n_points,
                   uint64_t* cost_out, uint16_t* arg_out, uint8_t* miss, hipStream_t st) {
  if (!n_points) return hipSuccess;
  static_assert(kIndexFan == 8, "a group of siblings is eight lanes and a byte of a ballot; node indices shift by 3 bits per level");
  return launch_checked(lookup_kernel, dim3((n_points + kLookupPoints - 1) / kLookupPoints, 2), dim3(256), st, g,
                        LookupLists{{lists[0], lists[1]}}, (const uint4*)points, vols, n_points, cost_out, arg_out, miss);
}

}  // namespace mrl
