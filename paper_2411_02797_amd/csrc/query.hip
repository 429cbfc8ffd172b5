// Batched lookup of call paths in a canonical tree: the analysis API's step that reads
// the metrics of the tree nodes on the call paths a search matched (Design,
// "Performance Analyzer", "Analysis API").
//
// A query path q is a node iff it is a prefix of some distinct full path.  With the
// full paths sorted, the first path p_i >= q is the only candidate that can start
// with q first; if it does, q is node (i, |q|) of p_i's chain, id = base_i + |q| -
// lcp_i - 1 (|q| > lcp_i holds, else p_{i-1} would start with q and be >= q).
//
// Two ways to find i:
//   - the prefix index (kept with the tree once built): every node (i, l), the depth-l
//     prefix of the path p_i that created it, under a 64-bit hash of that prefix; a query
//     hashes its frames, probes, and verifies every candidate frame by frame against the
//     stored path, so a lookup costs a few round trips;
//   - binary search over the sorted paths (when the index cannot be allocated).
#include <algorithm>

#include "common.h"

namespace cct {

namespace {

// four frames at a 4-byte-aligned address (one 16-byte load)
struct __attribute__((aligned(4))) Frames4 {
  uint32_t f[4];
};

// compare the path at canonical position i with query frames qf[0..ql), both known to
// agree on their first k0 frames: sign and common prefix length.  The path's first frame
// and length come from one 16-byte record; four frames per step, then one at a time.
__device__ int cmp_path_query(const QueryArgs &a, int64_t i, const uint32_t *qf, int64_t ql, int64_t k0,
                              int64_t *lcp) {
  const PathRec *rec = a.sorted + i;
  const int64_t fs = rec->start, lp = rec->len;
  const uint32_t *pf = a.pframes + fs;
  const int64_t n = min(lp, ql);
  int64_t k = k0;
  for (; k + 4 <= n; k += 4) {
    const Frames4 x = *reinterpret_cast<const Frames4 *>(pf + k);
    const Frames4 y = *reinterpret_cast<const Frames4 *>(qf + k);
    if (x.f[0] != y.f[0] || x.f[1] != y.f[1] || x.f[2] != y.f[2] || x.f[3] != y.f[3]) break;
  }
  for (; k < n; ++k) {
    const uint32_t x = pf[k], y = qf[k];
    if (x != y) { *lcp = k; return x < y ? -1 : 1; }
  }
  *lcp = n;
  return lp < ql ? -1 : (lp > ql ? 1 : 0);
}

// ---- prefix index ----------------------------------------------------------------------
// Hash of a prefix f_0 .. f_{l-1}: the sum of position-dependent terms (a repeated cycle of
// frames does not cancel: both factors move with the position), then a murmur3-style
// finalizer with the length.  Sums extend frame by frame, so one scan along a path gives
// the hash of every prefix.  Correctness never depends on it: every match is verified.
struct PrefixFactors {
  uint32_t x, y;
};
__device__ inline PrefixFactors prefix_factors(uint32_t f, uint32_t k) {
  return {f + k * 0x9E3779B9u, ((f ^ 0x5BD1E995u) + k * 0x85EBCA6Bu) | 1u};
}
__device__ inline uint64_t prefix_term(uint32_t f, uint32_t k) {
  const PrefixFactors t = prefix_factors(f, k);
  return (uint64_t)t.x * t.y;
}
__device__ inline uint64_t prefix_key(uint64_t sum, uint64_t len, uint64_t mask) {
  uint64_t h = sum ^ (len * 0xD6E8FEB86659FD93ull);
  h ^= h >> 33;
  h *= 0xFF51AFD7ED558CCDull;
  h ^= h >> 33;
  h *= 0xC4CEB9FE1A85EC53ull;
  h ^= h >> 33;
  return (h & mask) | 1;  // never the empty key 0
}

__device__ inline uint64_t shfl_up_u64(uint64_t v, int o) {
  const uint32_t lo = __shfl_up((uint32_t)v, o), hi = __shfl_up((uint32_t)(v >> 32), o);
  return ((uint64_t)hi << 32) | lo;
}
__device__ inline uint64_t shfl_u64(uint64_t v, int src) {
  const uint32_t lo = __shfl((uint32_t)v, src), hi = __shfl((uint32_t)(v >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}

// One wave per canonical position i: lane k of a 64-frame step holds frame k; an inclusive
// scan of the terms gives the prefix sums; the path's new nodes (depths lcp_i + 1 .. len)
// are inserted by linear probing (a 64-bit CAS claims an empty key; equal keys of other
// nodes just probe on).  The table is at most half full, so every probe sequence ends.
__global__ __launch_bounds__(256) void query_index_kernel(QueryArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (i >= a.d) return;
  const int64_t fs = a.sorted[i].start, len = a.sorted[i].len;
  const int64_t L = a.sorted[i].lcp;
  const uint32_t *pf = a.pframes + fs;
  uint64_t carry = 0;
  for (int64_t k0 = 0; k0 < len; k0 += 64) {
    const int64_t k = k0 + lane;
    const uint64_t t = k < len ? prefix_term(pf[k], (uint32_t)k) : 0;
    uint64_t sc = t;
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t y = shfl_up_u64(sc, o);
      if (lane >= o) sc += y;
    }
    if (k < len && k + 1 > L) {
      const uint64_t key = prefix_key(carry + sc, (uint64_t)(k + 1), a.qhash_mask);
      uint64_t slot = key & a.qcap_mask;
      for (uint64_t probe = 0; probe <= a.qcap_mask; ++probe) {
        const unsigned long long old = atomicCAS((unsigned long long *)&a.qtab[2 * slot], 0ull,
                                                 (unsigned long long)key);
        if (old == 0) {
          a.qtab[2 * slot + 1] = ((uint64_t)(k + 1) << 32) | (uint64_t)i;
          break;
        }
        slot = (slot + 1) & a.qcap_mask;
      }
    }
    carry += shfl_u64(sc, 63);
  }
}

// record of canonical position i: all that a lookup needs of the path, in one 32-byte load
__global__ void sorted_paths_kernel(QueryArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.d) return;
  const uint32_t p = a.order[i];
  PathRec r;
  r.start = a.pstart[p];
  r.len = a.plen[p];
  r.lcp = a.lcp[i];
  r.base = (int64_t)(1 + a.scan_out[i * (1 + a.m)]);
  r.pad = 0;
  a.sorted[i] = r;
}

// ---- lookup through the index -----------------------------------------------------------
// Several lanes per query.  A lookup is a chain of dependent reads (offsets, frames, table
// entry, path record, stored frames, sums), so its time is the number of queries in flight; with
// one lane per query every 16-byte load of a wave touched 64 different lines, and the frames of
// a query were read in a serial loop.  L lanes read 4 L consecutive frames per instruction, keep
// up to V pieces of them in registers for the comparison with the stored path (longer queries
// read theirs again), and meet by cross-lane moves.  1,048,576 queries of 68 frames on average
// in a tree of 4.2 million nodes: one lane per query 694 us; sixteen lanes 268 us (too few
// queries in flight); four lanes 218 us; eight lanes 214 us with three pieces at 7 waves per
// SIMD, 219 us with four at 6, 222 us with two at 8.  It moves about 0.9 GB (queries, stored
// frames, a table line and two rows of sums per query), 4.2 TB/s.
// Short queries leave most of eight lanes' work to padding, so a batch takes the lanes that its
// mean length fills: 32 frames on four lanes of two pieces, 16 frames on two lanes of two where
// no lane has more than two metrics to fetch.  Microseconds for 8,000,000 queries of 1,
// 8 and 16 frames (2 metrics, 40,000 nodes): eight lanes 877, 973 and 999, four 480, 541 and
// 565, two 311, 360 and 383, one lane with a serial loop 304, 497 and 774; for 1,000,000 of 32
// frames in 4,000,000 nodes 186 on eight lanes and 130 on four.  Two lanes lose to four from 4
// metrics on (1,000,000 queries of 8 frames in 4,000,000 nodes: 113 on four, 130 on two; with 8
// metrics 132 and 243) and from 20 frames on.

// sum over the L (2, 4 or 8) lanes of a query, on all of them
template <int L>
__device__ inline uint64_t sum_lanes(uint64_t v) {
#define CCT_DPP_ADD(ctrl)                                                                                    \
  {                                                                                                          \
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, ctrl, 0xF, 0xF, true);          \
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), ctrl, 0xF, 0xF, true);  \
    v += ((uint64_t)hi << 32) | lo;                                                                          \
  }
  CCT_DPP_ADD(0xB1)              // quad_perm 1,0,3,2
  if (L > 2) CCT_DPP_ADD(0x4E)   // quad_perm 2,3,0,1
  if (L > 4) CCT_DPP_ADD(0x141)  // row_half_mirror: the other quad of the eight lanes
#undef CCT_DPP_ADD
  return v;
}

// frames k .. k + 3 of a query of n frames (those below n; the others are unspecified).
// avail: frames readable from its first one (to the end of the batch).
template <class Int>
__device__ inline Frames4 query_frames(const uint32_t *qf, Int k, Int n, Int avail) {
  Frames4 v = {{0u, 0u, 0u, 0u}};
  if (k + 4 <= avail) {
    if (k < n) v = *reinterpret_cast<const Frames4 *>(qf + k);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (k + j < n) v.f[j] = qf[k + j];
  }
  return v;
}

// kQueryLanes lanes per query, kQueryVecs 16-byte pieces of it per lane
template <int kQueryLanes, int kQueryVecs>
__device__ inline void query_one(const QueryArgs &a, int64_t q, int lane) {
  constexpr int kQueryStep = 4 * kQueryLanes;          // frames per piece of the query's lanes
  constexpr int kQueryKeep = kQueryStep * kQueryVecs;  // frames held in registers
  int g = lane % kQueryLanes;
  // (opaque to the compiler here, or it keeps every lane-derived constant of the pieces
  // in registers across the queries: 138 VGPRs instead of 72)
  asm volatile("" : "+v"(g));
  const int64_t qs = a.qoff[q], qe = a.qoff[q + 1], ql = qe - qs, avail = a.qn_frames - qs;
  const uint32_t *qf = a.qfr + qs;
  int64_t id = -1;
  if (ql == 0) {
    id = 0;  // the empty path is the root
  } else {
    // the frames kept in registers, in 32-bit arithmetic (n of them)
    const int n = (int)min(ql, (int64_t)kQueryKeep), av = (int)min(avail, (int64_t)kQueryKeep);
    Frames4 f[kQueryVecs];
    uint64_t sum = 0;
#pragma unroll
    for (int c = 0; c < kQueryVecs; ++c) f[c] = query_frames<int>(qf, c * kQueryStep + 4 * g, n, av);
#pragma unroll
    for (int c = 0; c < kQueryVecs; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = c * kQueryStep + 4 * g + j;
        const PrefixFactors t = prefix_factors(f[c].f[j], (uint32_t)k);
        sum += (uint64_t)(k < n ? t.x : 0u) * t.y;
      }
    for (int64_t k0 = kQueryKeep; k0 < ql; k0 += kQueryStep) {
      const Frames4 x = query_frames<int64_t>(qf, k0 + 4 * g, ql, avail);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t k = k0 + 4 * g + j;
        sum += k < ql ? prefix_term(x.f[j], (uint32_t)k) : 0ull;
      }
    }
    const uint64_t key = prefix_key(sum_lanes<kQueryLanes>(sum), (uint64_t)ql, a.qhash_mask);
    uint64_t slot = key & a.qcap_mask;
    // probe from the query's key: an empty slot ends the sequence; an entry with the same
    // key and length is checked frame by frame against its path
    for (uint64_t probe = 0; probe <= a.qcap_mask; ++probe) {
      const ulonglong2 e = *reinterpret_cast<const ulonglong2 *>(a.qtab + 2 * slot);
      if (e.x == 0) break;
      if (e.x == key && (int64_t)(e.y >> 32) == ql) {
        const PathRec rec = a.sorted[(uint32_t)e.y];
        const uint32_t *pf = a.pframes + rec.start;
        uint32_t differ = (int64_t)rec.len < ql;
        if (!differ) {
          // (a stored path is padded to whole 16-frame blocks and holds the query's
          // frames, so a piece that starts below n stays in it)
          Frames4 p[kQueryVecs];
#pragma unroll
          for (int c = 0; c < kQueryVecs; ++c) {
            const int k = c * kQueryStep + 4 * g;
            p[c] = *reinterpret_cast<const Frames4 *>(pf + (k < n ? k : 0));
          }
#pragma unroll
          for (int c = 0; c < kQueryVecs; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) differ |= c * kQueryStep + 4 * g + j < n ? p[c].f[j] ^ f[c].f[j] : 0u;
          for (int64_t k0 = kQueryKeep; k0 < ql; k0 += kQueryStep) {
            const int64_t k = k0 + 4 * g;
            const Frames4 x = query_frames<int64_t>(qf, k, ql, avail);
            const Frames4 y = *reinterpret_cast<const Frames4 *>(pf + (k < ql ? k : 0));
#pragma unroll
            for (int j = 0; j < 4; ++j) differ |= k + j < ql ? x.f[j] ^ y.f[j] : 0u;
          }
        }
        if (((__ballot(differ != 0) >> (lane - g)) & ((1u << kQueryLanes) - 1)) == 0) {
          id = rec.base + ql - (int64_t)rec.lcp - 1;
          if (id >= a.u || ql <= (int64_t)rec.lcp) {  // cannot happen on a canonical tree
            if (g == 0) atomicOr(a.err + 1, 2ull);
            id = -1;
          }
          break;
        }
      }
      slot = (slot + 1) & a.qcap_mask;
    }
  }
  if (g == 0) a.node_ids[q] = id;
  for (int j = g; j < a.m; j += kQueryLanes) {
    const uint64_t x = a.qexcl && id >= 0 ? a.excl[id * a.m + j] : 0, y = a.qincl && id >= 0 ? a.incl[id * a.m + j] : 0;
    if (a.qexcl) a.qexcl[q * a.m + j] = x;
    if (a.qincl) a.qincl[q * a.m + j] = y;
  }
}

template <int L, int V>
__global__ __launch_bounds__(256, 7) void query_kernel(QueryArgs a) {
  if (*a.err) return;  // malformed offsets (query_check_kernel): nothing is written
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x / L;
  for (int64_t q = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / L; q < a.q; q += stride)
    query_one<L, V>(a, q, lane);
}

// ---- lookup by binary search ------------------------------------------------------------
// node id of the query by binary search over the sorted paths, or -1: the first i with
// path_i >= q.  llo and lhi: common prefix of q with the path below the range (path_{lo-1})
// and with the path above it (path_hi), 0 for the open ends.  Every path between two paths
// that share a prefix with q shares it too (paths with a given prefix are consecutive in
// lexicographic order), so a comparison can skip min(llo, lhi) frames.
__device__ int64_t search_lookup(const QueryArgs &a, const uint32_t *qf, int64_t ql) {
  int64_t lo = 0, hi = a.d, llo = 0, lhi = 0;
  int64_t l;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (cmp_path_query(a, mid, qf, ql, min(llo, lhi), &l) < 0) {
      lo = mid + 1;
      llo = l;
    } else {
      hi = mid;
      lhi = l;
    }
  }
  int64_t id = -1;
  if (lo < a.d) {
    l = lhi;  // lo = hi < D: set by the comparison with path_hi, which measured its prefix
    const PathRec rec = a.sorted[lo];
    if (l == ql) id = rec.base + ql - (int64_t)rec.lcp - 1;
    if (id >= a.u || (l == ql && ql <= (int64_t)rec.lcp)) {  // cannot happen on a canonical tree
      atomicOr(a.err + 1, 2ull);
      id = -1;
    }
  }
  return id;
}

// The query batch's offsets, checked before any output is written: err bit 0 when they
// do not start at 0, decrease, leave the frames or do not end at n_frames.
__global__ void query_check_kernel(QueryArgs a) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= a.q) return;
  const int64_t qs = a.qoff[q], qe = a.qoff[q + 1];
  if (qs < 0 || qe < qs || qe > a.qn_frames || (q == 0 && qs != 0) || (q + 1 == a.q && qe != a.qn_frames))
    atomicOr(a.err, 1ull);
}

__global__ void query_search_kernel(QueryArgs a) {
  if (*a.err) return;  // malformed offsets: nothing is written
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= a.q) return;
  const int64_t qs = a.qoff[q], qe = a.qoff[q + 1];
  const int64_t id = qe == qs ? 0 : search_lookup(a, a.qfr + qs, qe - qs);  // (the empty path is the root)
  a.node_ids[q] = id;
  for (int j = 0; j < a.m; ++j) {
    if (a.qexcl) a.qexcl[q * a.m + j] = id >= 0 ? a.excl[id * a.m + j] : 0;
    if (a.qincl) a.qincl[q * a.m + j] = id >= 0 ? a.incl[id * a.m + j] : 0;
  }
}

}  // namespace

void launch_sorted_paths(const QueryArgs &a, hipStream_t s) {
  if (a.d > 0) hipLaunchKernelGGL(sorted_paths_kernel, dim3((unsigned)((a.d + 255) / 256)), dim3(256), 0, s, a);
}

void launch_query_index(const QueryArgs &a, hipStream_t s) {
  if (a.d > 0) hipLaunchKernelGGL(query_index_kernel, dim3((unsigned)((a.d * 64 + 255) / 256)), dim3(256), 0, s, a);
}

void launch_query_check(const QueryArgs &a, hipStream_t s) {
  if (a.q > 0) hipLaunchKernelGGL(query_check_kernel, dim3((unsigned)((a.q + 255) / 256)), dim3(256), 0, s, a);
}

void launch_query(const QueryArgs &a, hipStream_t s) {
  if (a.q <= 0) return;
  if (a.qtab) {
    // (a launch holds fewer than 2^32 work items: larger batches loop)
    const bool brief = a.qn_frames <= 16 * a.q && a.m <= 3, medium = a.qn_frames <= 32 * a.q;
    const int lanes = brief ? 2 : medium ? 4 : 8;
    const dim3 blocks((unsigned)std::min<int64_t>((a.q * lanes + 255) / 256, 1 << 22));
    if (brief) hipLaunchKernelGGL((query_kernel<2, 2>), blocks, dim3(256), 0, s, a);
    else if (medium) hipLaunchKernelGGL((query_kernel<4, 2>), blocks, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((query_kernel<8, 3>), blocks, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL(query_search_kernel, dim3((unsigned)((a.q + 255) / 256)), dim3(256), 0, s, a);
  }
}

}  // namespace cct
