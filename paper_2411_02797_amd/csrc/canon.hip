// Canonical tree from the D distinct full paths (path store + exclusive sums).
//
// The paper's tree is a pointer structure with no node numbering (Design,
// "Profiler", "Calling Context Tree"); this library numbers nodes by the unsigned
// lexicographic rank of their root path.  With the D distinct full paths sorted
// lexicographically (p_0 < p_1 < ...) and lcp_i the length of the longest common
// prefix of p_{i-1} and p_i (lcp_0 = 0):
//   - path i contributes exactly the nodes p_i[0..l) for l in (lcp_i, len_i] (its
//     chain), which are new and, in id order, follow every node of the earlier
//     paths; so node ids are base_i + (l - lcp_i - 1) with base_i = 1 + sum of the
//     chain lengths (len - lcp) of earlier paths, and U = 1 + sum of all of them;
//   - the parent of a chain's first node is the node p_i[0..lcp_i), created by the
//     largest c < i with lcp_c < lcp_i (previous smaller value); every other chain
//     node's parent is the node before it;
//   - the paths through node (i, l) are exactly p_i .. p_{e-1}, e the first j > i
//     with lcp_j < l (next smaller value), and since a metric is added at the last
//     node of its path and then counted at every node up to the root (Design,
//     "Profiler", "Calling Context Tree"), inclusive(i, l) = S[e] - S[i] with S the
//     exclusive prefix sum of the per-path sums in sorted order (mod 2^64);
//   - exclusive(i, len_i) = the sums of path i, every other node has none (the empty
//     path, which sorts first, puts its sums on the root).
// Every step is a sort, a scan or an O(log D) search: the number of kernel launches
// does not grow with the tree depth.
#include <algorithm>

#include "common.h"

namespace cct {

namespace {

constexpr uint32_t kInf = 0xFFFFFFFFu;
constexpr int kMergeItems = 8;     // outputs per thread per merge pass
constexpr int kScanRows = 1024;    // rows per scan block

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// the order is not strictly increasing: the host sorts again by exact comparisons.  (A fast
// order that failed breaks nearly every pair, and atomics on one word wait for each other, 11 ns
// each: 400,000 paths 570 us in lcp_kernel when every pair raised the flag, 99 us so.)
__device__ inline void violated(unsigned long long *u_out) {
  if (*(volatile unsigned long long *)&u_out[1] == 0) atomicOr(&u_out[1], 1ull);
}

__device__ inline u32x4 ld4(const uint32_t *p) { return *(const u32x4 *)p; }

// Exact comparison of two stored paths: returns <0, 0, >0 and their lcp.  Starts are
// 16-frame aligned and tails are padded, so 16-byte loads never leave a path's slot.
__device__ int path_cmp_exact(const CanonArgs &a, uint32_t x, uint32_t y, uint32_t from, uint32_t *lcp) {
  const uint32_t lx = a.plen[x], ly = a.plen[y];
  const uint32_t *px = a.pframes + a.pstart[x], *py = a.pframes + a.pstart[y];
  const uint32_t n = min(lx, ly);
  for (uint32_t q = from & ~15u; q < n; q += 16) {
    u32x4 vx[4], vy[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) { vx[c] = ld4(px + q + 4 * c); vy[c] = ld4(py + q + 4 * c); }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t k = q + 4 * c + e;
        if (k < n && vx[c][e] != vy[c][e]) {
          *lcp = k;
          return vx[c][e] < vy[c][e] ? -1 : 1;
        }
      }
    }
  }
  *lcp = n;
  return lx < ly ? -1 : (lx > ly ? 1 : 0);
}

// Comparison accelerated by checkpoint hashes (prefix hashes every 16 frames): skip
// to the first 16-frame block whose prefix hashes differ, then compare frames
// there.  A hash collision can only make this answer wrong, never loop or fault;
// the exact verification after the sort catches any resulting misorder.
__device__ bool path_less(const CanonArgs &a, uint32_t x, uint32_t y) {
  if (x == kInf) return false;
  if (y == kInf) return true;
  uint32_t l;
  if (a.exact) return path_cmp_exact(a, x, y, 0, &l) < 0;
  const uint32_t lx = a.plen[x], ly = a.plen[y];
  const int64_t sx = a.pstart[x], sy = a.pstart[y];
  const uint32_t n = min(lx, ly), nb = n / kStoreAlign;
  const uint64_t *cx = a.pcp + sx / kStoreAlign, *cy = a.pcp + sy / kStoreAlign;
  uint32_t b = 0;
  for (; b + 4 <= nb; b += 4) {
    uint64_t hx[4], hy[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) { hx[c] = cx[b + c]; hy[c] = cy[b + c]; }
    int c = 0;
    while (c < 4 && hx[c] == hy[c]) ++c;
    if (c < 4) { b += c; goto found; }
  }
  for (; b < nb; ++b)
    if (cx[b] != cy[b]) break;
found:
  {
    // first differing frame is in block b (or in the partial block past nb)
    const int r = path_cmp_exact(a, x, y, b * kStoreAlign, &l);
    if (l < min(n, (b + 1) * kStoreAlign) || b >= nb) return r < 0;
    return path_cmp_exact(a, x, y, 0, &l) < 0;  // hashes differed, frames did not
  }
}

// Sort order: (gap, path) when a gap array is given (the new paths of a merge), else
// the path alone.
__device__ inline bool key_less(const CanonArgs &a, uint32_t x, uint32_t y) {
  if (x == kInf) return false;
  if (y == kInf) return true;
  if (a.gap) {
    const uint32_t gx = a.gap[x - a.id0], gy = a.gap[y - a.id0];
    if (gx != gy) return gx < gy;
  }
  return path_less(a, x, y);
}

// ---- sort -------------------------------------------------------------------------
// A large merge orders its new paths in one of two ways, and gap_kernel's samples say which:
// launches of the other way end at once.
enum When : int { kAlways = 0, kFewGaps = 1, kManyGaps = 2 };
__device__ inline bool skipped(const CanonArgs &a, When when) {
  return when != kAlways && (a.u_out[2] >= a.few_gaps) != (when == kFewGaps);
}

// Block-local bitonic sort by path, or by (gap, path).
__global__ __launch_bounds__(512) void sort_block_kernel(CanonArgs a, uint32_t *out, When when) {
  __shared__ uint32_t key[kSortBlock];
  if (skipped(a, when)) return;
  if (!a.gap) stamp(a.stamps + kStampOrder);
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * kSortBlock;
  for (int i = tid; i < kSortBlock; i += 512) key[i] = base + i < a.d ? (uint32_t)(a.id0 + base + i) : kInf;
  __syncthreads();
  for (int k = 2; k <= kSortBlock; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      const int i = 2 * j * (tid / j) + (tid % j), l = i + j;
      const uint32_t x = key[i], y = key[l];
      // ascending where (i & k) == 0: swap if y < x; else swap if x < y
      const bool up = (i & k) == 0;
      const bool swap = key_less(a, up ? y : x, up ? x : y);
      __syncthreads();
      if (swap) { key[i] = y; key[l] = x; }
      __syncthreads();
    }
  }
  for (int i = tid; i < kSortBlock; i += 512)
    if (base + i < a.d) out[base + i] = key[i];
}

// Block-local order of a merge's new paths by (gap, path): sixteen lanes share a path and
// count the block's paths before it, four gaps per load; the paths themselves are compared
// only within a gap.  The counts need no barrier and no second pass, so a block of 1024
// takes a few round trips: 10 us, where a bitonic sort took 40 us comparing paths in every
// step, and 26 us ordering the gaps first (55 steps on one CU).  With one block (place), the
// paths go straight to their place in the new order.
constexpr int kNewLanes = 16;
__global__ __launch_bounds__(256) void sort_new_kernel(CanonArgs a, uint32_t *out, uint32_t *gsorted,
                                                       uint32_t *place, uint32_t *placed, When when) {
  if (skipped(a, when)) return;
  const int g = threadIdx.x % kNewLanes;
  const int64_t j = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kNewLanes;
  if (j >= a.d) return;
  const int64_t base = j / kSortBlock * kSortBlock;
  const int n = (int)(a.d - base < kSortBlock ? a.d - base : kSortBlock), own = (int)(j - base);
  const uint32_t x = (uint32_t)(a.id0 + j), gx = a.gap[j];
  uint32_t before = 0;
  for (int k0 = 4 * g; k0 < n; k0 += 4 * kNewLanes) {
    const u32x4 v = ld4(a.gap + base + k0);  // (the array is padded to whole blocks)
    uint32_t tie = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = k0 + e < n && k0 + e != own;
      before += in && v[e] < gx;
      tie |= in && v[e] == gx ? 1u << e : 0u;
    }
    for (; tie; tie &= tie - 1)
      before += path_less(a, (uint32_t)(a.id0 + base + k0 + __builtin_ctz(tie)), x);
  }
#pragma unroll
  for (int o = kNewLanes / 2; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
  if (g != 0) return;
  gsorted[base + before] = gx;
  if (place) {
    place[gx + before] = x;
    a.lcp[gx + before] = kInf;  // not known yet
    placed[j] = 1;
  } else {
    out[base + before] = x;
  }
}

// The sorted blocks of a merge's new paths (ids, gaps bgap) into one order: a path's rank is
// its position in its block plus, for every other block, the paths there before it, found by
// binary search.  Sixteen lanes share a path, a block each: the search by gap needs 4-byte
// loads only; where the block holds paths in the same gap, a second one compares paths.
// Every block costs each path the same searches, so past kRankBlocks the merge passes, which
// grow with the logarithm of the number of blocks, are used instead: merges of new paths in
// 50,000 gaps by ranks and by passes, 34,000 296 and 431 us, 60,000 385 and 485, 66,000 424 and
// 535, 100,000 622 and 619, 130,000 823 and 682 (the line stays below 98 blocks because paths that
// share a gap cost the ranks more).
constexpr int64_t kRankBlocks = 64;
// Counting and ranking compare paths for every pair that shares a gap, so where most new paths
// lie in few gaps (a new phase of the program, a merge into a tree of few paths) their work grows
// with the square.  Past kCountBlocks gap_kernel's samples decide between them and the
// comparison sort of the blocks with merge passes; whichever is not needed costs its empty
// launches (8 of them, 11 to 18 us).  The share of neighbours in one gap from which the sort is
// taken falls as the blocks grow more (launch_merge_order).  New paths of 24 frames in 6 gaps, merged
// by counting and by sorting: 33,000 603 and 617 us, 60,000 1,000 and 653, 150,000 1,678 and
// 1,026; in 65 gaps: 33,000 385 and about 580, 60,000 700 and 616, 150,000 1,113 and 934; 200 gaps:
// 60,000 592 and about 640, 150,000 1,016 and 888.  Paths that share 100 frames, in few gaps: 26,000
// 824 and 863 us, 33,000 1,382 and 953, 60,000 2,188 and 1,056.
constexpr int64_t kCountBlocks = 26;
__global__ __launch_bounds__(256) void rank_new_kernel(CanonArgs a, const uint32_t *ids, const uint32_t *bgap,
                                                       uint32_t *gsorted, uint32_t *place, uint32_t *placed,
                                                       When when) {
  if (skipped(a, when)) return;
  const int g = threadIdx.x % kNewLanes;
  const int64_t j = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kNewLanes;
  if (j >= a.d) return;
  const uint32_t x = ids[j], gx = bgap[j];
  const int64_t own = j / kSortBlock, nb = (a.d + kSortBlock - 1) / kSortBlock;
  uint32_t before = g == 0 ? (uint32_t)(j - own * kSortBlock) : 0u;
  for (int64_t b = g; b < nb; b += kNewLanes) {
    if (b == own) continue;
    const uint32_t *gb = bgap + b * kSortBlock, *ib = ids + b * kSortBlock;
    const int n = (int)(a.d - b * kSortBlock < kSortBlock ? a.d - b * kSortBlock : kSortBlock);
    int lo = 0, hi = n;  // first path of the block with a gap >= gx
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (gb[mid] < gx) lo = mid + 1; else hi = mid;
    }
    if (lo < n && gb[lo] == gx) {
      int end = n, from = lo;  // its paths in gap gx: [lo, end)
      while (from < end) {
        const int mid = (from + end) >> 1;
        if (gb[mid] <= gx) from = mid + 1; else end = mid;
      }
      while (lo < end) {
        const int mid = (lo + end) >> 1;
        if (path_less(a, ib[mid], x)) lo = mid + 1; else end = mid;
      }
    }
    before += (uint32_t)lo;
  }
#pragma unroll
  for (int o = kNewLanes / 2; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
  if (g == 0) {
    gsorted[before] = gx;
    place[gx + before] = x;
    a.lcp[gx + before] = kInf;  // not known yet
    placed[x - a.id0] = 1;
  }
}

__global__ __launch_bounds__(256) void merge_pass_kernel(CanonArgs a, const uint32_t *src, uint32_t *dst,
                                                         int64_t run, When when) {
  if (skipped(a, when)) return;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t o0 = t * kMergeItems;
  if (o0 >= a.d) return;
  const int64_t pair = o0 / (2 * run), pb = pair * 2 * run;
  const int64_t la = min(run, a.d - pb), lb = max((int64_t)0, min(run, a.d - pb - run));
  const uint32_t *A = src + pb, *B = src + pb + la;
  const int64_t dgl = o0 - pb;
  int64_t lo = max((int64_t)0, dgl - lb), hi = min(dgl, la);
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (key_less(a, A[mid], B[dgl - 1 - mid])) lo = mid + 1; else hi = mid;
  }
  int64_t ia = lo, ib = dgl - lo;
  const int64_t cnt = min((int64_t)kMergeItems, la + lb - dgl);
  for (int64_t k = 0; k < cnt; ++k) {
    bool take_a;
    if (ia >= la) take_a = false;
    else if (ib >= lb) take_a = true;
    else take_a = !key_less(a, B[ib], A[ia]);
    dst[o0 + k] = take_a ? A[ia++] : B[ib++];
  }
}

// A merge's new paths: gap[j] = number of old paths (in their sorted order) below
// new path d_old + j.  Sixteen lanes search for one new path: each step compares it with
// 16 old paths that cut the remaining range into 17 parts (a 17-ary search), so the
// answer takes about log_17(d_old) rounds of path comparisons instead of log_2(d_old)
// (each comparison is a chain of dependent loads).
constexpr int kGapLanes = 16, kGapSample = 16;
__global__ __launch_bounds__(256) void gap_kernel(CanonArgs a, const uint32_t *old_order, int64_t d_old, uint32_t *gap,
                                                  uint32_t *ids, uint32_t *bgap, uint32_t *gsorted, uint32_t *placed) {
  stamp(a.stamps + kStampOrder);
  const int lane = threadIdx.x & 63, g = lane % kGapLanes, g0 = lane - g;
  const int64_t j = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kGapLanes;
  const bool active = j < a.d - d_old;
  const uint32_t x = (uint32_t)(d_old + (active ? j : 0));
  // old_order[0, lo) are below x, old_order[hi, d_old) are not
  int64_t lo = 0, hi = active ? d_old : 0;
  for (;;) {
    const int64_t n = hi - lo;
    if (!__any(n > 0)) break;
    // pivot of this lane: every position when the range is at most 16 long, else the
    // 16 cuts into 17 parts (distinct and increasing for n >= 17)
    const int64_t pv = n <= kGapLanes ? lo + g : lo + (n * (g + 1)) / (kGapLanes + 1);
    const bool below = n > 0 && pv < hi && path_less(a, old_order[pv], x);
    const uint32_t m = (uint32_t)(__ballot(below) >> g0) & ((1u << kGapLanes) - 1);
    const int c = __popc(m);  // the pivots below x are a prefix (the old order is sorted)
    const int64_t p_lo = __shfl((long long)pv, g0 + (c > 0 ? c - 1 : 0), 64);
    const int64_t p_hi = __shfl((long long)pv, g0 + (c < kGapLanes ? c : kGapLanes - 1), 64);
    if (n > 0) {
      if (n <= kGapLanes) {
        lo += c;
        hi = lo;
      } else {
        const int64_t nlo = c > 0 ? p_lo + 1 : lo, nhi = c < kGapLanes ? p_hi : hi;
        lo = nlo;
        hi = nhi;
      }
    }
  }
  // every 16th workgroup counts the neighbours among its waves' four paths that share a gap
  if (a.few_gaps && blockIdx.x % kGapSample == 0) {
    const uint32_t next = __shfl((uint32_t)lo, (g0 + kGapLanes) & 63, 64);
    const uint64_t same = __ballot(active && g == 0 && g0 + kGapLanes < 64 && next == (uint32_t)lo);
    if (lane == 0 && same) atomicAdd(&a.u_out[2], (unsigned long long)__popcll(same));
  }
  if (active && g == 0) {
    gap[j] = (uint32_t)lo;
    // a hash collision can make two paths claim one place of an order below.  The place no path
    // claims then keeps these values: in a block's order a path and its gap, so that what reads
    // them stays in bounds, though that path then comes twice; in the whole order a gap that
    // none has.  A path that lost its place in either is not marked as placed.
    ids[j] = x;
    bgap[j] = (uint32_t)lo;
    gsorted[j] = kInf;
    placed[j] = 0;
  }
}

// Placement: the r-th new path (sorted by gap, then path) goes after its gap's old
// paths and the r new paths before it; old path i goes after the new paths whose
// gap is <= i.  Where no new path comes between old paths i - 1 and i, their LCP is the one
// the tree keeps (lcp: kInf elsewhere): only pairs with a new path are compared again.
__global__ __launch_bounds__(256) void place_new_kernel(const uint32_t *B, int64_t n_new, int64_t d_old,
                                                        const uint32_t *gap, uint32_t *gsorted, uint32_t *dst, uint32_t *lcp,
                                                        uint32_t *placed, CanonArgs a, When when) {
  if (skipped(a, when)) return;
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_new) return;
  const uint32_t x = B[r];
  const uint32_t g = gap[x - d_old];
  gsorted[r] = g;
  dst[g + r] = x;
  lcp[g + r] = kInf;  // not known yet
  placed[x - d_old] = 1;
}
__global__ __launch_bounds__(256) void place_old_kernel(const uint32_t *A, int64_t d_old, const uint32_t *gsorted,
                                                        const uint32_t *placed, int64_t n_new, const uint32_t *old_lcp,
                                                        uint32_t *dst, uint32_t *lcp, unsigned long long *u_out,
                                                        unsigned long long *stamps) {
  if (n_new == 0) stamp(stamps + kStampOrder);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // Comparisons that collided hashes misled (neither of two paths before the other, or three in
  // a cycle) can give one rank to two paths.  The new paths' order is whole iff every path was
  // placed, every rank taken (as many ranks as paths: each once) and the gaps ascend; then all
  // places of the order are written, and neighbours whose LCP is not kept are compared.
  // Otherwise nothing below is believed and the host sorts again by exact comparisons.
  if (i < n_new) {
    const uint32_t g = gsorted[i];
    if (g == kInf || !placed[i] || (i > 0 && gsorted[i - 1] > g)) violated(u_out);
  }
  if (i >= d_old) return;
  int64_t lo = 0, hi = n_new;  // new paths with gap <= i
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)gsorted[mid] <= i) lo = mid + 1; else hi = mid;
  }
  dst[i + lo] = A[i];
  lcp[i + lo] = i > 0 && !(lo > 0 && (int64_t)gsorted[lo - 1] == i) ? old_lcp[i] : kInf;
}
// ---- exact verification, lcp, sums, scan rows ------------------------------------------------
// Eight lanes per pair of neighbours: a step compares 64 frames of both, two 16-byte loads
// per lane and path, and the first lane with a difference holds the LCP.  With one lane per
// pair the longest paths of a wave set its time, eight dependent 16-byte loads per 16
// frames.  Now, with the scan's block sums, level 1 of the minima and the sums' fold in the
// same pass (they were two launches more): 14,444 paths of up to 2,500 frames 191 -> 33 us,
// 149,201 paths of 256 to 512 frames 86 -> 61 us (their frames at 8 TB/s from the caches),
// 154,413 paths of 72 frames on average 24 -> 25 us.  Sixteen lanes with one load: 21, 66
// and 36 us; four lanes with four: 36, 61 and 23 us.
constexpr int kLcpLanes = 8;
constexpr int kLcpPieces = 2;                        // 16-byte loads per lane, path and step
constexpr int kLcpPer = 256 / kLcpLanes;             // positions per workgroup and round
constexpr uint32_t kLcpPiece = 4 * kLcpLanes;        // frames per piece
static_assert(kLcpPer % 16 == 0, "whole entries of level 1 of the minima per workgroup and round");

// lcp of position i (every lane of the position's group gets it); u_out[1] if the two paths
// are not strictly increasing
__device__ inline uint32_t lcp_at(const CanonArgs &a, int64_t i, uint32_t p, uint32_t len, int64_t start, int lane) {
  const int g = lane % kLcpLanes;
  if (i == 0) return 0;
  uint32_t q = a.order[i - 1];
  if (q >= (uint64_t)a.d) q = 0;
  const uint32_t lq = a.plen[q], n = min(lq, len);
  const uint32_t *pq = a.pframes + a.pstart[q], *pp = a.pframes + start;
  bool less = lq < len;  // the order of the two if they agree on n frames
  uint32_t l = n;
  bool done = false;
  for (uint32_t k0 = 0; k0 < n && !done; k0 += kLcpPiece * kLcpPieces) {
    // (starts are 16-frame aligned and tails are padded: a lane whose first frame is
    // below n stays in both paths' slots)
    u32x4 x[kLcpPieces], y[kLcpPieces];
#pragma unroll
    for (int v = 0; v < kLcpPieces; ++v) {
      const uint32_t k = k0 + v * kLcpPiece + 4 * g, at = k < n ? k : 0;
      x[v] = ld4(pq + at);
      y[v] = ld4(pp + at);
    }
#pragma unroll
    for (int v = 0; v < kLcpPieces; ++v) {
      const uint32_t k = k0 + v * kLcpPiece + 4 * g;
      uint32_t e = 8;  // this lane's first difference: frame, and whether x is the smaller
#pragma unroll
      for (int c = 3; c >= 0; --c)
        if (k + c < n && x[v][c] != y[v][c]) e = 2 * c + (x[v][c] < y[v][c] ? 1 : 0);
      const uint32_t found = (uint32_t)(__ballot(e < 8) >> (lane - g)) & ((1u << kLcpLanes) - 1);
      if (found && !done) {
        const int f = __builtin_ctz(found);
        const uint32_t ef = __shfl(e, lane - g + f, 64);
        l = k0 + v * kLcpPiece + 4 * f + (ef >> 1);
        less = ef & 1;
        done = true;
      }
    }
  }
  if (!less && g == 0) violated(a.u_out);  // not strictly increasing
  return l;
}

// A workgroup's consecutive positions lie in one block of the scan, whose sums they meet
// in LDS first (one atomic per column), and fill whole entries of level 1 of the minima.
__global__ __launch_bounds__(256) void lcp_kernel(CanonArgs a) {
  __shared__ uint32_t ls[kLcpPer];
  __shared__ uint64_t rows[kLcpPer][9];
  const int C = 1 + a.m, lane = threadIdx.x & 63, g = lane % kLcpLanes, r = threadIdx.x / kLcpLanes;
  stamp(a.stamps + kStampNodes);
  // what the merge order knows holds in a whole order only: a place that no path claimed keeps
  // what the memory held before, so once the order is known to have one every pair is compared
  const bool known = a.lcp_known && a.u_out[1] == 0;
  // levels of the minima from 3 up are met by atomics in the next kernel
  if (blockIdx.x == 0)
    for (int v = 3; v < a.min_levels; ++v)
      for (int64_t k = threadIdx.x; k < a.min_n[v]; k += blockDim.x) a.mins[v][k] = kInf;
  for (int64_t i0 = (int64_t)blockIdx.x * kLcpPer; i0 <= a.d; i0 += (int64_t)gridDim.x * kLcpPer) {
    const int64_t i = i0 + r;
    uint32_t l = kInf;  // (past the last position)
    CanonRec rc{};
    if (i == a.d) l = 0;
    if (i < a.d) {
      // an order from a misleading hash may hold entries that are not path ids: they raise
      // the flag and read as path 0 here and in the kernels after this one
      uint32_t p = a.order[i];
      const bool bad = p >= (uint64_t)a.d;
      if (bad) p = 0;
      const uint32_t len = a.plen[p], sl = a.pslot[p];
      rc.start = a.pstart[p];
      l = known && i > 0 ? a.lcp[i] : kInf;  // (position 0 has LCP 0 whatever the memory holds)
      if (l > len) l = lcp_at(a, i, p, len, rc.start, lane);
      rc.len = len;
      rc.lcp = l;
      if (bad && g == 0) {
        violated(a.u_out);
        a.order[i] = 0;
      }
      // the path's sums after the batch: every path sits at one position of a good order,
      // so this pass folds each path's batch sums into its old ones, into the fresh array
      // (a bad order's leftovers are overwritten when the corrected order comes through)
      for (int c = g; c < C; c += kLcpLanes) {
        uint64_t v = (uint64_t)(len - l);
        if (c > 0) {
          const int64_t at = (int64_t)p * a.m + c - 1;
          v = a.delta[(uint64_t)sl * a.m + c - 1] + (p < (uint64_t)a.d_old ? a.old_sums[at] : 0);
          a.psums[at] = v;
        }
        a.scan_in[i * C + c] = v;
        rows[r][c] = v;
      }
    } else {
      for (int c = g; c < C; c += kLcpLanes) rows[r][c] = 0;
    }
    if (g == 0) {
      ls[r] = l;
      if (i <= a.d) a.lcp[i] = l;
      if (i < a.d) a.rec[i] = rc;
    }
    __syncthreads();
    if ((int)threadIdx.x < C) {
      uint64_t t = 0;
#pragma unroll
      for (int k = 0; k < kLcpPer; ++k) t += rows[k][threadIdx.x];
      if (t) atomicAdd((unsigned long long *)&a.scan_blk[i0 / kScanRows * C + threadIdx.x], (unsigned long long)t);
    } else if (threadIdx.x >= 64 && threadIdx.x < 64 + kLcpPer / 16) {
      const int e = (int)threadIdx.x - 64;
      uint32_t t = kInf;
#pragma unroll
      for (int k = 0; k < 16; ++k) t = min(t, ls[16 * e + k]);
      if (i0 / 16 + e < a.min_n[1] && a.min_levels > 1) a.mins[1][i0 / 16 + e] = t;
    }
    __syncthreads();
  }
}

// ---- multi-column exclusive scan (uint64, mod 2^64) -------------------------------------
__device__ inline uint64_t shfl_up_u64(uint64_t v, int o) {
  uint32_t lo = __shfl_up((uint32_t)v, o, 64), hi = __shfl_up((uint32_t)(v >> 32), o, 64);
  return ((uint64_t)hi << 32) | lo;
}

__global__ __launch_bounds__(256) void scan_reduce_kernel(const uint64_t *in, int64_t rows, int C, uint64_t *blk) {
  __shared__ uint64_t part[4];
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kScanRows;
  for (int c = blockIdx.y; c < C; c += gridDim.y) {
    uint64_t s = 0;
    for (int64_t r = r0 + tid; r < min(rows, r0 + kScanRows); r += 256) s += in[r * C + c];
    for (int o = 32; o > 0; o >>= 1) {
      uint32_t lo = __shfl_xor((uint32_t)s, o, 64), hi = __shfl_xor((uint32_t)(s >> 32), o, 64);
      s += ((uint64_t)hi << 32) | lo;
    }
    if ((tid & 63) == 0) part[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) blk[blockIdx.x * C + c] = part[0] + part[1] + part[2] + part[3];
    __syncthreads();
  }
}

// exclusive scan of the block sums in place; totals into out row `rows`
__global__ __launch_bounds__(256) void scan_blocks_kernel(uint64_t *blk, int64_t nblk, int C, uint64_t *out,
                                                          int64_t rows) {
  __shared__ uint64_t part[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int c = 0; c < C; ++c) {
    uint64_t carry = 0;
    for (int64_t b0 = 0; b0 < nblk; b0 += 256) {
      const int64_t b = b0 + tid;
      const uint64_t v = b < nblk ? blk[b * C + c] : 0;
      uint64_t x = v;
      for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = shfl_up_u64(x, o);
        if (lane >= o) x += y;
      }
      if (lane == 63) part[wave] = x;
      __syncthreads();
      uint64_t before = carry;
      for (int w = 0; w < wave; ++w) before += part[w];
      if (b < nblk) blk[b * C + c] = before + x - v;
      const uint64_t tot = part[0] + part[1] + part[2] + part[3];
      __syncthreads();
      carry += tot;
    }
    if (tid == 0) out[rows * C + c] = carry;
  }
}

// direct: blk holds the raw block sums (not scanned), and each block adds up the sums of
// the blocks before it itself (at most kScanDirectBlocks of them); the last block also
// writes the totals row.  Otherwise blk holds their exclusive scan (scan_blocks_kernel).
constexpr int64_t kScanDirectBlocks = 4096;

__global__ __launch_bounds__(256) void scan_final_kernel(const uint64_t *in, int64_t rows, int C, const uint64_t *blk,
                                                         uint64_t *out, int direct) {
  __shared__ uint64_t part[4];
  __shared__ uint64_t pre;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kScanRows + tid * 4;
  for (int c = blockIdx.y; c < C; c += gridDim.y) {
    if (direct) {  // sum of the earlier blocks' sums of column c
      uint64_t x = 0;
      for (int64_t j = tid; j < (int64_t)blockIdx.x; j += 256) x += blk[j * C + c];
      for (int o = 32; o > 0; o >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)x, o, 64), hi = __shfl_xor((uint32_t)(x >> 32), o, 64);
        x += ((uint64_t)hi << 32) | lo;
      }
      if (lane == 0) part[wave] = x;
      __syncthreads();
      if (tid == 0) pre = part[0] + part[1] + part[2] + part[3];
      __syncthreads();
    }
    uint64_t v[4], s = 0;
    for (int k = 0; k < 4; ++k) {
      v[k] = r0 + k < rows ? in[(r0 + k) * C + c] : 0;
      s += v[k];
    }
    uint64_t x = s;
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t y = shfl_up_u64(x, o);
      if (lane >= o) x += y;
    }
    if (lane == 63) part[wave] = x;
    __syncthreads();
    const uint64_t base = direct ? pre : blk[blockIdx.x * C + c];
    uint64_t run = base + x - s;
    for (int w = 0; w < wave; ++w) run += part[w];
    for (int k = 0; k < 4; ++k) {
      if (r0 + k < rows) out[(r0 + k) * C + c] = run;
      run += v[k];
    }
    if (direct && blockIdx.x == gridDim.x - 1 && tid == 0) out[rows * C + c] = base + part[0] + part[1] + part[2] + part[3];
    __syncthreads();
  }
}

// ---- scan of the canonical rows, upper levels of the minima -----------------------------
// Workgroup (b, y) writes the exclusive prefix sums of columns y, y + gridDim.y, ... of
// rows [1024 b, 1024 b + 1024).  scan_blk holds the sums of every 1024 rows (lcp_kernel):
// each workgroup adds up those before it (direct), or they are scanned already.  The
// workgroups with y = 0 also build level 2 of the minima and meet in the levels above.
__global__ __launch_bounds__(256) void canon_scan_kernel(CanonArgs a, int direct) {
  __shared__ uint64_t part[4], pre[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, C = 1 + a.m;
  const int64_t b = blockIdx.x, r0 = b * kScanRows + tid * 4;
  if (blockIdx.y == 0 && tid < 64 && a.min_levels > 2) {
    const int64_t k = b * (kScanRows / 16) + tid;
    uint32_t t = k < a.min_n[1] ? a.mins[1][k] : kInf;
    for (int o = 32; o > 0; o >>= 1) t = min(t, (uint32_t)__shfl_xor(t, o, 64));
    if (tid == 0) {
      a.mins[2][b] = t;
      int64_t at = b;
      for (int v = 3; v < a.min_levels; ++v) {
        at >>= 6;
        atomicMin(&a.mins[v][at], t);
      }
    }
  }
  for (int c = blockIdx.y; c < C; c += gridDim.y) {
    uint64_t v[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = r0 + k < a.d ? a.scan_in[(r0 + k) * C + c] : 0;
      s += v[k];
    }
    uint64_t x = 0;  // this thread's share of the sums of the earlier blocks
    if (direct)
      for (int64_t j = tid; j < b; j += 256) x += a.scan_blk[j * C + c];
    for (int o = 32; o > 0; o >>= 1) {
      const uint32_t lo = __shfl_xor((uint32_t)x, o, 64), hi = __shfl_xor((uint32_t)(x >> 32), o, 64);
      x += ((uint64_t)hi << 32) | lo;
    }
    uint64_t y = s;
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t z = shfl_up_u64(y, o);
      if (lane >= o) y += z;
    }
    if (lane == 0) pre[wave] = x;
    if (lane == 63) part[wave] = y;
    __syncthreads();
    uint64_t run = (direct ? pre[0] + pre[1] + pre[2] + pre[3] : a.scan_blk[b * C + c]) + y - s;
    for (int w = 0; w < wave; ++w) run += part[w];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      // (row D holds the totals: every row before it is in this block or an earlier one)
      if (r0 + k <= a.d) a.scan_out[(r0 + k) * C + c] = run;
      run += v[k];
    }
    __syncthreads();
  }
}

// ---- range minima of lcp over [0, D] (lcp[D] = 0 is the sentinel) --------------------
// The searches below look at sixteen entries at a time (four 16-byte loads in flight
// together): most answers lie in the entries next to the start, one round trip away.
// (A table of every power of two took two launches to build, 17 words per path, and a
// search of it two dependent 4-byte loads per doubling of the distance.)

// Positions fit 32 bits (a tree has fewer than 2^32 - 2 nodes, and every path but the
// empty one a node of its own); not-found is kInf.

// bit k: p[k] < t, for sixteen entries at a 64-byte aligned address
__device__ inline uint32_t below16(const uint32_t *p, uint32_t t) {
  u32x4 v[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = ld4(p + 4 * c);
  uint32_t m = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) m |= v[c][e] < t ? 1u << (4 * c + e) : 0u;
  return m;
}
// first entry from k to the last one of its group of w (16 or 64; last: the level's last
// entry) below t
__device__ inline uint32_t first_below(const uint32_t *lv, uint32_t k, uint32_t w, uint32_t last, uint32_t t) {
  const uint32_t end = min(k | (w - 1), last);
  for (uint32_t c = k & ~15u;; c += 16) {
    uint32_t m = below16(lv + c, t);
    if (c < k) m &= ~0u << (k - c);
    if (m) {
      const uint32_t f = c + (uint32_t)__builtin_ctz(m);
      return f <= end ? f : kInf;  // (past the end: padding)
    }
    if (end - c < 16) return kInf;
  }
}
// last entry from the first one of k's group of w up to k below t
__device__ inline uint32_t last_below(const uint32_t *lv, uint32_t k, uint32_t w, uint32_t t) {
  for (uint32_t c = k & ~15u;; c -= 16) {
    uint32_t m = below16(lv + c, t);
    if (k - c < 15) m &= (2u << (k - c)) - 1;
    if (m) return c + 31 - (uint32_t)__builtin_clz(m);
    if ((c & (w - 1)) == 0) return kInf;
  }
}

// first j >= s with lcp[j] < t (exists for s <= D: lcp[D] = 0 < t for t >= 1): up through
// the levels to the first entry that holds such a position, then down to it
__device__ inline uint32_t next_smaller(const CanonArgs &a, uint32_t s, uint32_t t) {
  uint32_t k = s, w = 16;
  int v = 0;
  for (;;) {
    const uint32_t f = first_below(a.mins[v], k, w, (uint32_t)a.min_n[v] - 1, t);
    if (f != kInf) { k = f; break; }
    k = k / w + 1;
    w = 64;
    if (++v == a.min_levels || k >= (uint64_t)a.min_n[v]) return (uint32_t)a.d;
  }
  while (v > 0) {
    k *= w = --v == 0 ? 16 : 64;
    k = first_below(a.mins[v], k, w, (uint32_t)a.min_n[v] - 1, t);
    if (k == kInf) return (uint32_t)a.d;
  }
  return k;
}
// largest j <= s with lcp[j] < t (exists for s >= 0: lcp[0] = 0 < t for t >= 1), the same
// search towards smaller indices
__device__ inline uint32_t prev_smaller(const CanonArgs &a, uint32_t s, uint32_t t) {
  uint32_t k = s, w = 16;
  int v = 0;
  for (;;) {
    const uint32_t f = last_below(a.mins[v], k, w, t);
    if (f != kInf) { k = f; break; }
    k /= w;
    w = 64;
    if (k-- == 0 || ++v == a.min_levels) return 0;
  }
  while (v > 0) {
    w = --v == 0 ? 16 : 64;
    k = (uint32_t)min((uint64_t)k * w + w - 1, (uint64_t)a.min_n[v] - 1);
    k = last_below(a.mins[v], k, w, t);
    if (k == kInf) return 0;
  }
  return k;
}

__device__ inline uint64_t node_base(const CanonArgs &a, int64_t i) { return 1 + a.scan_out[i * (1 + a.m)]; }

// chain parent of each path and the node -> path map.  The order is checked only after
// these kernels: if it is not a permutation (a misleading hash can repeat a path), the
// node count can exceed u_max, so nodes past it are not written and the order-violation
// flag is raised (the host then sorts again by exact comparisons).
__global__ void chain_kernel(CanonArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.d) return;
  const uint32_t L = a.lcp[i];
  uint32_t par = 0;
  if (L > 0) {
    const int64_t c = prev_smaller(a, i - 1, L);
    par = (uint32_t)(node_base(a, c) + L - a.lcp[c] - 1);
  }
  a.chain_parent[i] = par;
  const uint64_t b = node_base(a, i);
  const uint32_t cnt = a.rec[i].len - L;
  if (b + cnt > (uint64_t)a.u_max) {
    violated(a.u_out);
    return;
  }
  if (cnt == 0) return;
  // the 64-node windows whose first node lies on this path (window 0 starts at node 1,
  // past the root)
  if (b == 1) a.win_path[0] = (uint32_t)i;
  for (uint64_t w = (b + 63) / 64; w <= (b + cnt - 1) / 64; ++w) a.win_path[w] = (uint32_t)i;
}

// One wave per window of 64 consecutive nodes.  The kernel is a chain of dependent loads
// (window's first path, bases of its 64 paths, a path's record, frame, end of the subtree,
// sums at the end), so the next window's first two are requested a window ahead, a path's
// fields come from one 16-byte record, and the M sums of a row are requested together (M is
// a template parameter).  7 waves per SIMD (72 VGPRs; 64 for 8 waves spill, 1 to 9 us
// slower); from 5 metrics on 5 are asked for (the LDS rows, 1 KB and 4 KB per metric, leave room for
// 7, 6, 5 and 4 workgroups).  The node arrays are written with non-temporal stores: nothing here
// reads them, and what they would evict from the caches is read (this kernel's rows, the next
// call's frames).  A first reader finds less of them in the caches, but a build with its first
// reader is no slower for it: build alone, with the first filter, with the view and with the
// export, about 10 million nodes of 2 metrics 772, 856, 1,461 and 930 us, with ordinary stores 817, 909,
// 1,507 and 961; about 4.5 million 556, 631, 945 and 655 against 560, 633, 942 and 652.  4,222,948 nodes of 2 metrics 114
// -> 81 us (2.5 TB/s of arrays written), 4.57 million of 4 metrics 149 -> 107 us (3.4), 4.0
// million of 8 metrics 166 -> 95 us (6.1).
template <int M>
__global__ __launch_bounds__(256, M <= 4 ? 7 : 5) void emit_kernel(CanonArgs a) {
  // a wave's 64 consecutive nodes stage their excl and incl rows in LDS, then write each
  // array's 64 M words as one contiguous stretch
  constexpr int C = 1 + M;
  __shared__ uint64_t stage[2][256 * M];
  __shared__ uint32_t emit_mark[256];  // per wave: window position -> path offset
  const int lane = threadIdx.x & 63, w0 = __builtin_amdgcn_readfirstlane(threadIdx.x - lane);
  uint64_t *sx = stage[0] + w0 * M, *si = stage[1] + w0 * M;
  // (bounded by u_max, as in chain_kernel: past it the order is not a permutation)
  const int64_t U_all = (int64_t)(1 + a.scan_out[a.d * C]);
  const int64_t U = U_all < a.u_max ? U_all : a.u_max;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.u_out[0] = (unsigned long long)U;
    if (U_all > a.u_max) violated(a.u_out);
  }
  uint32_t *mark = emit_mark + w0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const uint32_t d = (uint32_t)a.d;
  // (positions and node ids fit 32 bits; a wave's window and its first path are uniform)
  // first path of the window at `base` (window 0 holds only the root when there is no other
  // node: no path to look up), and the first node of path i
  auto window_path = [&](int64_t base) -> uint32_t {
    return __builtin_amdgcn_readfirstlane(base < U && (base > 0 || U > 1) ? a.win_path[base >> 6] : 0u);
  };
  auto first_node = [&](uint32_t i) -> uint32_t {
    return i < d ? 1 + (uint32_t)a.scan_out[(uint64_t)i * C] : kInf;
  };
  int64_t base = (int64_t)blockIdx.x * blockDim.x + w0;
  uint32_t i0 = window_path(base);
  uint32_t nb = first_node(i0 + lane);
  for (; base < U; base += stride) {
    const uint32_t b0 = (uint32_t)base, u = b0 + lane;
    const uint32_t i0_next = window_path(base + stride);
    // this window's paths: the one holding its first node and the 63 after it (every
    // path past the first has at least one node, so they cover the window); a node's
    // path is the last of them whose first node is at or before it
    if (i0 >= d && (base > 0 || U > 1)) {  // a window chain_kernel did not write (the order is not a permutation)
      if (lane == 0) violated(a.u_out);
      i0 = 0;
      nb = first_node(lane);
    }
    mark[lane] = 0;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    if (lane > 0 && nb >= b0 && nb - b0 < 64) mark[nb - b0] = (uint32_t)lane;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    uint32_t off = mark[lane];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(off, o, 64);
      if (lane >= o) off = max(off, y);
    }
    uint32_t b = __shfl(nb, (int)off, 64);
    const uint32_t nb_next = first_node(i0_next + lane);
    if (u == 0) {
      a.parent[0] = kInf;
      a.frame[0] = 0;
      a.depth[0] = 0;
      a.subend[0] = (uint32_t)U;
      const bool empty_path = d > 0 && a.rec[0].len == 0;
      for (int j = 0; j < M; ++j) {
        sx[j] = empty_path ? a.scan_out[C + 1 + j] : 0;
        si[j] = a.scan_out[a.d * C + 1 + j];
      }
    } else if (base + lane < U) {
      uint32_t i = i0 + off;
      if (i >= d || b > u) {  // (only when the order is not a permutation)
        violated(a.u_out);
        i = 0;
        b = first_node(0);
      }
      const CanonRec rc = a.rec[i];
      const uint32_t after = a.lcp[i + 1];
      uint32_t l = rc.lcp + 1 + (u - b);
      if (l > rc.len || u - b >= rc.len) {  // (only when the order is not a permutation)
        violated(a.u_out);
        l = rc.len;
      }
      const uint32_t fr = l ? a.pframes[rc.start + l - 1] : 0u;
      __builtin_nontemporal_store(u == b ? a.chain_parent[i] : u - 1, &a.parent[u]);
      __builtin_nontemporal_store(l, &a.depth[u]);
      const uint32_t e = i + 1 == d || l > after ? i + 1 : next_smaller(a, i + 2, l);
      __builtin_nontemporal_store(fr, &a.frame[u]);
      // the subtree is the paths i .. e-1 below depth l: ids up to the first node of path e
      const uint64_t *pi = a.scan_out + (uint64_t)i * C, *pe = a.scan_out + (uint64_t)e * C;
      __builtin_nontemporal_store((uint32_t)(1 + (uint32_t)pe[0]), &a.subend[u]);
      uint64_t from[M], to[M];  // the sums of the paths before i, before e
#pragma unroll
      for (int j = 0; j < M; ++j) {
        from[j] = pi[1 + j];
        to[j] = pe[1 + j];
      }
#pragma unroll
      for (int j = 0; j < M; ++j) si[lane * M + j] = to[j] - from[j];
      // the path's own sums at its last node (mostly the row just read: a path's last node
      // is most often a leaf)
      if (l == rc.len && e != i + 1) {
#pragma unroll
        for (int j = 0; j < M; ++j) to[j] = pi[C + 1 + j];
      }
#pragma unroll
      for (int j = 0; j < M; ++j) sx[lane * M + j] = l == rc.len ? to[j] - from[j] : 0;
    }
    // every lane's LDS writes before any lane's reads
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    const int words = (int)(U - base < 64 ? U - base : 64) * M;
#pragma unroll
    for (int q = 0; q < M; ++q) {
      const int k = 64 * q + lane;
      if (k < words) {
        __builtin_nontemporal_store(sx[k], &a.excl[base * M + k]);
        __builtin_nontemporal_store(si[k], &a.incl[base * M + k]);
      }
    }
    // every lane's reads before the next nodes' writes
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    i0 = i0_next;
    nb = nb_next;
  }
}

// Array blockIdx.y: 16 bytes per lane and step where both ends allow it.  The copies are not
// read again here (non-temporal).
__global__ __launch_bounds__(256) void copy_kernel(CopyArgs a) {
  const uint32_t *src = a.src[blockIdx.y];
  uint32_t *dst = a.dst[blockIdx.y];
  const uint64_t n = a.words[blockIdx.y], t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x,
                 stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t done = 0;
  if ((((uintptr_t)src | (uintptr_t)dst) & 15) == 0) {
    done = n / 4 * 4;
    for (uint64_t i = t; i < n / 4; i += stride)
      __builtin_nontemporal_store(__builtin_nontemporal_load((const u32x4 *)src + i), (u32x4 *)dst + i);
  }
  for (uint64_t i = done + t; i < n; i += stride) dst[i] = src[i];
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

namespace {
// merge passes over blocks of kSortBlock sorted ids: the sorted list, in one of the buffers
uint32_t *merge_blocks(const CanonArgs &a, uint32_t *src, uint32_t *dst, When when, hipStream_t s) {
  for (int64_t run = kSortBlock; run < a.d; run *= 2) {
    hipLaunchKernelGGL(merge_pass_kernel, dim3(blocks_for((a.d + kMergeItems - 1) / kMergeItems, 256)), dim3(256),
                       0, s, a, src, dst, run, when);
    uint32_t *t = src; src = dst; dst = t;
  }
  return src;
}
}  // namespace

void launch_sort(CanonArgs &a, hipStream_t s) {
  if (a.d <= 0) return;
  hipLaunchKernelGGL(sort_block_kernel, dim3(blocks_for(a.d, kSortBlock)), dim3(512), 0, s, a, a.order, kAlways);
  uint32_t *sorted = merge_blocks(a, a.order, a.order_tmp, kAlways, s);
  if (sorted != a.order) {
    a.order_tmp = a.order;
    a.order = sorted;
  }
}

void launch_merge_order(CanonArgs &a, const uint32_t *old_order, const uint32_t *old_lcp, int64_t d_old,
                        uint32_t *scratch, hipStream_t s) {
  const int64_t n_new = a.d - d_old;
  const int64_t room = (n_new + kSortBlock - 1) / kSortBlock * kSortBlock;
  uint32_t *gap = scratch, *gsorted = scratch + room, *placed = scratch + 3 * room;
  uint32_t *dst = a.order;
  a.lcp_known = 1;
  if (n_new > 0) {
    const int64_t nb = room / kSortBlock;
    uint32_t *src = a.order, *tmp = a.order_tmp, *bgap = scratch + 2 * room;
    const dim3 lanes(blocks_for(n_new * kNewLanes, 256)), blocks((unsigned)nb), paths(blocks_for(n_new, 256));
    CanonArgs r = a;  // the new ids by (gap, path)
    r.d = n_new;
    r.id0 = d_old;
    r.gap = gap;
    const bool either = nb > kCountBlocks;  // counting or comparing, as the gaps say
    if (either) {
      // the share of neighbours in one gap at which sorting pays: see kCountBlocks (a sampled
      // workgroup compares 12 pairs; beyond kRankBlocks only the blocks' order is in question)
      const int64_t pairs = (int64_t)blocks_for(blocks_for(n_new * kGapLanes, 256), kGapSample) * 12;
      r.few_gaps = a.few_gaps = (uint64_t)std::max<int64_t>(1, pairs / (nb <= 40 ? 4 : nb <= 48 ? 16 : nb <= kRankBlocks ? 64 : 128));
    }
    hipLaunchKernelGGL(gap_kernel, dim3(blocks_for(n_new * kGapLanes, 256)), dim3(256), 0, s, a, old_order, d_old, gap,
                       nb > 1 ? src : tmp, bgap, gsorted, placed);
    hipLaunchKernelGGL(sort_new_kernel, lanes, dim3(256), 0, s, r, src, nb > 1 ? bgap : gsorted,
                       nb > 1 ? (uint32_t *)nullptr : dst, placed, either ? kManyGaps : kAlways);
    if (nb > 1) dst = tmp;
    if (nb > 1 && nb <= kRankBlocks)
      hipLaunchKernelGGL(rank_new_kernel, lanes, dim3(256), 0, s, r, src, bgap, gsorted, dst, placed,
                         either ? kManyGaps : kAlways);
    if (either) {
      const When when = nb <= kRankBlocks ? kFewGaps : kAlways;
      int passes = 0;
      for (int64_t run = kSortBlock; run < n_new; run *= 2) ++passes;
      // (up to kRankBlocks the sorted list has to end where rank_new_kernel read its blocks)
      uint32_t *from = when == kFewGaps && passes % 2 ? tmp : src;
      hipLaunchKernelGGL(sort_block_kernel, blocks, dim3(512), 0, s, r, from, kFewGaps);
      uint32_t *sorted = merge_blocks(r, from, from == src ? tmp : src, when, s);
      dst = sorted == src ? tmp : src;
      hipLaunchKernelGGL(place_new_kernel, paths, dim3(256), 0, s, sorted, n_new, d_old, gap, gsorted, dst, a.lcp, placed,
                         r, when);
    }
  }
  hipLaunchKernelGGL(place_old_kernel, dim3(blocks_for(std::max(d_old, n_new), 256)), dim3(256), 0, s, old_order,
                     d_old, gsorted, placed, n_new, old_lcp, dst, a.lcp, a.u_out, a.stamps);
  a.order_tmp = dst == a.order ? a.order_tmp : a.order;
  a.order = dst;
}

void launch_scan(const uint64_t *in, int64_t rows, int C, uint64_t *blk, uint64_t *out, hipStream_t s) {
  if (rows > 0) {
    const int64_t nblk = (rows + kScanRows - 1) / kScanRows;
    const int direct = nblk <= kScanDirectBlocks ? 1 : 0;
    // few blocks: the columns side by side as well (each then reads the rows for itself)
    const unsigned cols = nblk <= 256 ? (unsigned)C : 1u;
    hipLaunchKernelGGL(scan_reduce_kernel, dim3((unsigned)nblk, cols), dim3(256), 0, s, in, rows, C, blk);
    if (!direct) hipLaunchKernelGGL(scan_blocks_kernel, dim3(1), dim3(256), 0, s, blk, nblk, C, out, rows);
    hipLaunchKernelGGL(scan_final_kernel, dim3((unsigned)nblk, cols), dim3(256), 0, s, in, rows, C, blk, out, direct);
  } else {
    (void)hipMemsetAsync(out, 0, sizeof(uint64_t) * C, s);
  }
}

void launch_copy(const CopyArgs &a, hipStream_t s) {
  uint64_t most = 1;
  for (int i = 0; i < a.n; ++i) most = std::max(most, a.words[i]);
  const unsigned grid = (unsigned)std::min<uint64_t>((most + 1023) / 1024, 4096);
  hipLaunchKernelGGL(copy_kernel, dim3(grid, a.n), dim3(256), 0, s, a);
}

int64_t min_level_words(int64_t n, CanonArgs &a) {
  int64_t words = 0, k = n;
  a.min_levels = 1;
  a.min_n[0] = n;
  while (k > (a.min_levels == 1 ? 16 : 64) && a.min_levels < 6) {  // until one group is left
    k = a.min_levels == 1 ? (k + 15) / 16 : (k + 63) / 64;
    a.min_n[a.min_levels++] = k;
    words += (k + 15) / 16 * 16;
  }
  return words;
}
void set_min_levels(CanonArgs &a, uint32_t *words) {
  a.mins[0] = a.lcp;
  for (int v = 1; v < a.min_levels; ++v) {
    a.mins[v] = words;
    words += (a.min_n[v] + 15) / 16 * 16;
  }
}

void launch_canon(const CanonArgs &a, hipStream_t s) {
  const int C = 1 + a.m;
  const int64_t n = a.d + 1;
  // (a launch holds fewer than 2^32 work items: more positions loop)
  hipLaunchKernelGGL(lcp_kernel, dim3(std::min(blocks_for(n, kLcpPer), 1u << 22)), dim3(256), 0, s, a);
  const int64_t nblk = (n + kScanRows - 1) / kScanRows;
  const int direct = nblk <= kScanDirectBlocks ? 1 : 0;
  if (!direct)
    hipLaunchKernelGGL(scan_blocks_kernel, dim3(1), dim3(256), 0, s, a.scan_blk, nblk, C, a.scan_out, a.d);
  // few blocks: the columns side by side as well (each then reads the rows for itself)
  hipLaunchKernelGGL(canon_scan_kernel, dim3((unsigned)nblk, nblk <= 256 ? C : 1), dim3(256), 0, s, a, direct);
  if (a.d > 0) hipLaunchKernelGGL(chain_kernel, dim3(blocks_for(a.d, 256)), dim3(256), 0, s, a);
  switch (a.m) {
#define CCT_EMIT_CASE(M)                                                                      \
  case M:                                                                                     \
    hipLaunchKernelGGL(emit_kernel<M>, dim3(a.grid_nodes), dim3(256), 0, s, a);               \
    break;
    CCT_EMIT_CASE(1) CCT_EMIT_CASE(2) CCT_EMIT_CASE(3) CCT_EMIT_CASE(4)
    CCT_EMIT_CASE(5) CCT_EMIT_CASE(6) CCT_EMIT_CASE(7) CCT_EMIT_CASE(8)
#undef CCT_EMIT_CASE
    default: break;
  }
}

}  // namespace cct
