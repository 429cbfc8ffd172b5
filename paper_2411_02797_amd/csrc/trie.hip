// Lexicographic order of the distinct full paths through a trie of 16-frame blocks.
//
// The canonical node ids are the lexicographic ranks of the paths (the paper's tree
// has no ids; see canon.hip).  Sorting variable-length paths by comparison needs long
// chains of dependent memory reads (paths share long prefixes), so the rank of each
// path is computed instead:
//   - every path of the path store is a chain of blocks of 16 frames (the last one
//     possibly shorter).  A block node is a distinct prefix ending at a block
//     boundary or at a path's end; nodes are deduplicated by hashing (the 16-frame
//     checkpoint hashes the store already holds) and then verified exactly: a node's
//     occurrences must share the parent node and the block's frames, which proves by
//     induction over the depth that equal nodes are equal prefixes;
//   - siblings (nodes with the same parent) are ordered by their blocks (frames
//     compared as unsigned, a shorter block first when it is a prefix of the other);
//   - with count(X) the number of paths through node X, the paths before path p are
//     those that leave p's chain X_1 .. X_n at an earlier sibling of some X_k, plus
//     the paths ending exactly at some X_{k-1} (proper prefixes of p):
//       rank(p) = sum_k [ sum of count(S) over siblings S < X_k  +  ends(X_{k-1}) ].
// A failed verification (a hash collision) or an oversized sibling group raises a
// flag, and the caller falls back to the comparison sort; the order is in any case
// re-verified frame by frame before it is used.
#include "common.h"

namespace cct {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int kBlk = kStoreAlign;           // frames per block
constexpr int kLarge = 512;                 // larger sibling groups are split into buckets ...
constexpr int64_t kSmallTrie = 2048;        // ... unless the trie has no more blocks than this
// Largest bucket that is ordered by counting; beyond it the call fails over to the comparison sort.
// Builds of n paths of 20 frames that part in the first block, with 2,048, 4,096 and 8,192 here:
// n = 200,000 1.60, 0.80 and 0.80 ms; 300,000 1.72, 1.30 and 1.27; 400,000 2.12, 2.10 and 1.79;
// from 700,000 on a bucket passes all three (3.87 ms).
constexpr int kMaxBucket = 8192;
constexpr uint64_t kRootSeed = 0x5851F42D4C957F2Dull;
constexpr int kMaxBuckets = 256, kOversample = 2, kBucketTarget = 32;  // large groups (split_kernel)
constexpr int kFail = kTrieCtrFail;

__device__ inline void fail(const TrieArgs &a) { atomicOr(&a.ctr[kFail], 1ull); }

// block s of the store (frames [16 s, 16 s + 16)): its index k in its path, depth
// (prefix length at its end) and the path's length, from one word per block
struct BlockPos {
  uint32_t k, depth, len;
};
__device__ inline BlockPos block_pos(const TrieArgs &a, int64_t s) {
  const uint64_t w = a.bpos[s];
  BlockPos b;
  b.k = (uint32_t)w;
  b.len = (uint32_t)(w >> 32);
  b.depth = min((b.k + 1) * (uint32_t)kBlk, b.len);
  return b;
}
// frames in a node's block (1..16), from its depth
__device__ inline uint32_t block_frames(uint32_t depth) { return ((depth - 1) & (kBlk - 1)) + 1; }

// empty the node table; zero the bucket counts and the root's child count
__global__ void clear_kernel(TrieArgs a) {
  stamp(a.stamps + kStampOrder);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (int64_t)a.cap) a.tkey[i] = 0;
  if (i < a.large_cap * kMaxBuckets) { a.bcnt[i] = 0; a.bsum[i] = 0; }
  if (i == 0) a.hist[a.cap] = 0;
}

// positions of the store blocks of paths [0, d) (publish_kernel writes those of new paths)
__global__ void fill_kernel(TrieArgs a, int64_t d_old) {
  const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (d >= d_old) return;
  const uint32_t len = a.plen[d];
  if (len == 0) {
    a.ctr[kTrieCtrEmpty] = 1;  // the empty path ends at the root
    return;
  }
  const int64_t b0 = a.pstart[d] / kBlk, nb = (len + kBlk - 1) / kBlk;
  for (int64_t k = 0; k < nb; ++k) a.bpos[b0 + k] = make_bpos(len, (uint64_t)k);
}

// Node of every block: open addressing on the prefix hash (claimed by CAS).  A node's id is
// the store block that claimed it, its representative, so its frames are found without a
// lookup and per-node arrays are about as long as there are nodes; the counters that many
// blocks add to at once (link_kernel) are kept by table slot, which spreads the nodes of a
// chain, most counted together, over different cache lines.
__global__ __launch_bounds__(256) void insert_kernel(TrieArgs a) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= a.nblocks) return;
  a.nend[s] = 0;
  const BlockPos b = block_pos(a, s);
  uint64_t key;
  if (b.depth == (b.k + 1) * kBlk) {
    key = a.pcp[s];  // full block: the checkpoint hash of the prefix
  } else {           // a path's last, partial block: hash it onto the previous checkpoint
    const uint32_t *f = a.pframes + s * kBlk;
    uint64_t acc = 0;
    for (uint32_t i = 0; i < b.depth - b.k * kBlk; ++i) acc += frame_term(f[i], b.k * kBlk + i);
    key = finish_hash(acc + (b.k ? a.pcp[s - 1] : kRootSeed) * 0x9E3779B97F4A7C15ull, b.depth);
  }
  if (key == 0) key = 1;
  const uint64_t mask = a.cap - 1;
  uint64_t slot = key & mask;
  for (uint64_t step = 0; step < a.cap; ++step) {
    uint64_t cur = a.tkey[slot];
    if (cur == 0) {
      cur = atomicCAS((unsigned long long *)&a.tkey[slot], 0ull, (unsigned long long)key);
      if (cur == 0) {
        a.tval[slot] = (uint32_t)s;
        a.count[slot] = 0;
        a.hist[slot] = 0;
        a.oslot[s] = (uint32_t)slot;
        return;
      }
    }
    if (cur == key) {
      a.oslot[s] = (uint32_t)slot;
      return;
    }
    slot = (slot + 1) & mask;
  }
  a.oslot[s] = 0;
  fail(a);
}

// slots to node ids
__global__ __launch_bounds__(256) void resolve_kernel(TrieArgs a) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= a.nblocks) return;
  const uint32_t X = a.tval[a.oslot[s]];
  a.occ[s] = X < (uint64_t)a.nblocks ? X : 0u;  // (always, unless the call has failed)
}

// Verify every occurrence against its node's representative (same depth, same parent
// node, same frames), link parents, count children per parent, paths per node (summed
// in an LDS map per workgroup first: nodes near the root are on many paths) and path
// ends.
constexpr int kLinkThreads = 1024, kLinkMap = 8192;
constexpr uint32_t kMapEmpty = 0xFFFFFFFFu;

__global__ __launch_bounds__(kLinkThreads) void link_kernel(TrieArgs a) {
  __shared__ uint32_t mkey[kLinkMap];
  __shared__ uint32_t mval[kLinkMap];
  __shared__ uint32_t root_children;
  for (int i = threadIdx.x; i < kLinkMap; i += kLinkThreads) { mkey[i] = kMapEmpty; mval[i] = 0; }
  if (threadIdx.x == 0) root_children = 0;
  __syncthreads();
  const int64_t lo = (int64_t)blockIdx.x * a.nblocks / gridDim.x, hi = (int64_t)(blockIdx.x + 1) * a.nblocks / gridDim.x;
  for (int64_t s = lo + threadIdx.x; s < hi; s += kLinkThreads) {
    const BlockPos b = block_pos(a, s);
    const uint32_t X = a.occ[s];
    const int64_t rep = (int64_t)X;
    const uint32_t slot = a.oslot[s];
    const uint32_t P = b.k ? a.occ[s - 1] : (uint32_t)a.nblocks;
    // the representative links the node and takes its index among its siblings (the
    // root's children, many, take theirs with one LDS atomic per wave)
    const bool is_rep = rep == s, to_root = P == (uint32_t)a.nblocks;
    const uint64_t rm = __ballot(is_rep && to_root);
    if (rm) {
      const int lane = threadIdx.x & 63, leader = __builtin_ctzll(rm);
      uint32_t base = 0;
      if (lane == leader) base = atomicAdd(&root_children, (uint32_t)__popcll(rm));
      base = __shfl(base, leader, 64);
      // (workgroup << 22) | index among this workgroup's root children
      if (is_rep && to_root) a.cidx[X] = (blockIdx.x << 22) | (base + (uint32_t)__popcll(rm & ((1ull << lane) - 1)));
    }
    if (is_rep) {
      a.nparent[X] = P;
      if (!to_root) a.cidx[X] = atomicAdd(&a.hist[a.oslot[s - 1]], 1u);
    } else {
      // (a representative of the same depth has this block's index in its path, and so sits
      // at store block k or later)
      bool ok = block_pos(a, rep).depth == b.depth && rep >= (int64_t)b.k;
      if (ok) {
        const uint32_t RP = b.k ? a.occ[rep - 1] : (uint32_t)a.nblocks;
        ok = RP == P;
        if (ok) {
          const u32x4 *x = (const u32x4 *)(a.pframes + s * kBlk), *y = (const u32x4 *)(a.pframes + rep * kBlk);
          const uint32_t nf = b.depth - b.k * kBlk;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const u32x4 vx = x[c], vy = y[c];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if ((uint32_t)(4 * c + e) < nf && vx[e] != vy[e]) ok = false;
          }
        }
      }
      if (!ok) fail(a);
    }
    uint32_t h = hash32(slot) & (kLinkMap - 1);
    bool done = false;
    for (int t = 0; t < 16 && !done; ++t) {
      uint32_t cur = mkey[h];
      if (cur == kMapEmpty) cur = atomicCAS(&mkey[h], kMapEmpty, slot);
      if (cur == kMapEmpty || cur == slot) {
        atomicAdd(&mval[h], 1u);
        done = true;
      } else {
        h = (h + 1) & (kLinkMap - 1);
      }
    }
    if (!done) atomicAdd(&a.count[slot], 1u);
    if (b.depth == b.len) a.nend[X] = 1;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kLinkMap; i += kLinkThreads)
    if (mkey[i] != kMapEmpty) atomicAdd(&a.count[mkey[i]], mval[i]);
  // the root's children: this workgroup's block of indices (the root is one hot counter)
  if (threadIdx.x == 0)
    a.rootbase[blockIdx.x] = root_children ? atomicAdd(&a.hist[a.cap], root_children) : 0u;
}

// Room for every node's children among the positions: a group is a contiguous range, the
// order of the groups does not matter (ranks add up counts of siblings only), so each
// workgroup takes room for its nodes' groups with one atomic (all of it is the number of
// nodes, each being a child of one).  Groups too large to be ordered by counting are
// listed.  The counters move from table slots to node ids; store block `nblocks` stands for
// the root.
__device__ inline uint32_t node_count(const TrieArgs &a) { return (uint32_t)a.ctr[kTrieCtrNodes]; }
constexpr int kAllocThreads = 1024, kAllocPer = 4;  // 256 blocks a workgroup (one atomic each): 46 us for 766,000; 4096: 19 us
__global__ __launch_bounds__(kAllocThreads) void alloc_kernel(TrieArgs a) {
  __shared__ uint32_t wsum[kAllocThreads / 64], base;
  const uint64_t nb = (uint64_t)a.nblocks, i0 = (uint64_t)blockIdx.x * kAllocThreads * kAllocPer;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t n[kAllocPer], total = 0;
#pragma unroll
  for (int k = 0; k < kAllocPer; ++k) {
    const uint64_t P = i0 + (uint64_t)k * kAllocThreads + threadIdx.x;
    n[k] = 0;
    if (P == nb) {
      n[k] = a.hist[a.cap];
    } else if (P < nb && a.occ[P] == P) {
      const uint32_t slot = a.oslot[P];
      n[k] = a.hist[slot];
      a.ncount[P] = a.count[slot];
    }
    total += n[k];
  }
  uint32_t x = total;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int q = 0; q < kAllocThreads / 64; ++q) {
      const uint32_t c = wsum[q];
      wsum[q] = t;
      t += c;
    }
    base = t ? (uint32_t)atomicAdd(&a.ctr[kTrieCtrNodes], (unsigned long long)t) : 0u;
  }
  __syncthreads();
  uint32_t g0 = base + wsum[w] + x - total;
#pragma unroll
  for (int k = 0; k < kAllocPer; ++k) {
    if (!n[k]) continue;
    const uint64_t P = i0 + (uint64_t)k * kAllocThreads + threadIdx.x;
    a.gstart[P] = g0;
    a.nchild[P] = n[k];
    if (n[k] > (uint32_t)a.large) {
      const unsigned long long q = atomicAdd(&a.ctr[kTrieCtrLarge], 1ull);
      if ((int64_t)q < a.large_cap) {
        a.lists[q] = ((uint64_t)g0 << 32) | n[k];
        a.lgroup[P] = (uint32_t)q;
      } else {  // (cannot happen: large_cap groups of this size hold every node)
        fail(a);
      }
    }
    g0 += n[k];
  }
}

// Nodes grouped by parent: position = start of the parent's group + the node's index among
// its siblings; unit: the range of positions the node is ordered within (its group).
__global__ __launch_bounds__(256) void scatter_kernel(TrieArgs a) {
  const uint64_t X = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (X >= (uint64_t)a.nblocks || a.occ[X] != X) return;
  const uint32_t P = a.nparent[X], ci = a.cidx[X];
  const uint32_t c = P == (uint32_t)a.nblocks ? a.rootbase[ci >> 22] + (ci & ((1u << 22) - 1)) : ci;
  const uint32_t g0 = a.gstart[P];
  a.grouped[g0 + c] = (uint32_t)X;
  a.unit[g0 + c] = ((uint64_t)g0 << 32) | a.nchild[P];
}

// ---- sibling order ------------------------------------------------------------------
// A node's block as eight 64-bit words, two frames each, the first in the high half, so
// that comparing two blocks is comparing eight words; and its number of frames.  Frames
// past a block's end are zero in the store: two blocks that differ there differ in a word
// where the shorter one has the zero, which then decides as the length rule does; blocks
// equal in all words are ordered by their lengths.
struct BlockRow {
  uint64_t w[kBlk / 2];
  uint32_t nf;
};
__device__ inline void node_row(const TrieArgs &a, uint32_t X, BlockRow &r) {
  const u32x4 *p = (const u32x4 *)(a.pframes + (uint64_t)X * kBlk);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const u32x4 v = p[c];
    r.w[2 * c] = ((uint64_t)v[0] << 32) | v[1];
    r.w[2 * c + 1] = ((uint64_t)v[2] << 32) | v[3];
  }
  r.nf = block_frames(block_pos(a, X).depth);
}
typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
// LDS rows: kRowWords words each
constexpr int kRowWords = kBlk / 2;
__device__ inline void put_row(uint64_t *lds, uint8_t *nf, const BlockRow &r) {
#pragma unroll
  for (int c = 0; c < kRowWords; c += 2) {
    const u64x2 v = {r.w[c], r.w[c + 1]};
    *(u64x2 *)(lds + c) = v;
  }
  *nf = (uint8_t)r.nf;
}
// LDS row x < row y, without branches
__device__ inline bool row_less(const uint64_t *x, uint32_t nx, const BlockRow &y) {
  bool less = nx < y.nf;
#pragma unroll
  for (int c = kRowWords - 2; c >= 0; c -= 2) {
    const u64x2 v = *(const u64x2 *)(x + c);
    less = v[1] < y.w[c + 1] || (v[1] == y.w[c + 1] && less);
    less = v[0] < y.w[c] || (v[0] == y.w[c] && less);
  }
  return less;
}

// Groups of more than kLarge siblings are cut into ordered buckets: splitters from a
// sorted sample (2 per bucket, aiming at buckets of about 32), every member's bucket by
// binary search over the splitters, the group reordered by bucket; the buckets are then
// ordered like the smaller groups.
__device__ inline int buckets_for(uint32_t n) {
  int nb = 2;
  while (nb < kMaxBuckets && (uint32_t)nb * kBucketTarget < n) nb <<= 1;
  return nb;
}
__device__ inline uint64_t large_groups(const TrieArgs &a) {
  return min((uint64_t)a.ctr[kTrieCtrLarge], (uint64_t)a.large_cap);
}

// Sample -> splitters (node ids).  A workgroup stages the group's sample in LDS and ranks
// kSplitPer of its entries, a wave an entry, by counting the entries before it; an entry of
// even rank r > 0 is splitter r / 2 - 1.  Equal blocks (which siblings have only where a hash
// collision joined their parents) rank in the order of the sample, so that the ranks are a
// permutation and every splitter is written whatever the blocks hold: classify_kernel reads
// them as node ids.  The comparisons bound it, so they are spread over
// 32 workgroups.  (1,048,576 events: a bitonic sort of the sample in one workgroup 28 us,
// every thread counting for an entry by itself 107 us, eight workgroups with sixteen lanes
// an entry 21 us, 9 us so.)
constexpr int kSplitLanes = 64, kSplitThreads = 1024, kSplitPer = kSplitThreads / kSplitLanes;
constexpr int kSamples = kMaxBuckets * kOversample;
static_assert(kOversample == 2, "splitters are the entries of even rank");
__global__ __launch_bounds__(kSplitThreads) void split_kernel(TrieArgs a) {
  __shared__ uint64_t sb[kSamples][kRowWords];
  __shared__ uint8_t sn[kSamples];
  const uint64_t ng = large_groups(a);
  for (uint64_t g = blockIdx.y; g < ng; g += gridDim.y) {
    const uint64_t e = a.lists[g];
    const uint32_t start = (uint32_t)(e >> 32), n = (uint32_t)e;
    const int ns = buckets_for(n) * kOversample;
    if ((int)blockIdx.x * kSplitPer >= ns) continue;  // (the whole workgroup)
    for (int i = threadIdx.x; i < ns; i += kSplitThreads) {
      BlockRow r;
      node_row(a, a.grouped[start + (uint64_t)i * n / ns], r);
      put_row(sb[i], &sn[i], r);
    }
    __syncthreads();
    const int i = (int)blockIdx.x * kSplitPer + threadIdx.x / kSplitLanes, l = threadIdx.x % kSplitLanes;
    if (i < ns) {
      BlockRow y;
#pragma unroll
      for (int c = 0; c < kRowWords; ++c) y.w[c] = sb[i][c];
      y.nf = 2 * sn[i] + 1;  // (frames doubled: room for the order in the sample)
      uint32_t rank = 0;
      for (int j = l; j < ns; j += kSplitLanes)
        rank += j != i && row_less(sb[j], 2 * sn[j] + (j > i ? 2u : 0u), y);
#pragma unroll
      for (int o = kSplitLanes / 2; o > 0; o >>= 1) rank += __shfl_xor(rank, o, 64);
      if (l == 0 && rank > 0 && rank % kOversample == 0)
        a.spl[g * kMaxBuckets + rank / kOversample - 1] = a.grouped[start + (uint64_t)i * n / ns];
    }
    __syncthreads();
  }
}

// Every member of a large group: its bucket (number of splitters below it) and its index
// there (place), and the buckets' sizes and path counts.  Groups of more than kLarge siblings:
// at most two of them have members among kClassPer consecutive positions, the first and the
// last position's.
constexpr int kClassPer = 512;
static_assert(kClassPer <= kLarge, "at most two large groups in a workgroup's positions");
__global__ __launch_bounds__(kClassPer) void classify_kernel(TrieArgs a) {
  __shared__ uint64_t sb[2][kMaxBuckets][kRowWords];
  __shared__ uint8_t sn[2][kMaxBuckets];
  __shared__ uint32_t grp[2];
  const uint64_t nodes = node_count(a);
  const uint64_t lo = (uint64_t)blockIdx.x * kClassPer;
  if (lo >= nodes) return;
  const uint64_t p = lo + threadIdx.x, ng = large_groups(a);
  uint32_t X = 0, g = 0xFFFFFFFFu;
  if (p < nodes && (uint32_t)a.unit[p] > (uint32_t)a.large) {
    X = a.grouped[p];
    g = a.lgroup[a.nparent[X]];  // listed large group (an unlisted one has already failed the call)
    if ((uint64_t)g >= ng) g = 0xFFFFFFFFu;
  }
  const uint64_t last = min(lo + kClassPer, nodes) - 1;
  if (p == lo) grp[0] = g;
  if (p == last) grp[1] = g;
  __syncthreads();
  if (grp[0] == 0xFFFFFFFFu && grp[1] == 0xFFFFFFFFu) return;  // (large groups cover more positions than these)
  for (int h = 0; h < 2; ++h) {
    const uint32_t gh = grp[h];
    if (gh == 0xFFFFFFFFu || (h == 1 && gh == grp[0])) continue;
    const int nb = buckets_for((uint32_t)a.lists[gh]);
    for (int j = threadIdx.x; j < nb - 1; j += kClassPer) {
      BlockRow r;
      node_row(a, a.spl[gh * kMaxBuckets + j], r);
      put_row(sb[h][j], &sn[h][j], r);
    }
  }
  __syncthreads();
  if (g == 0xFFFFFFFFu) return;
  const int h = g == grp[0] ? 0 : 1;
  BlockRow y;
  node_row(a, X, y);
  int blo = 0, bhi = buckets_for((uint32_t)a.lists[g]) - 1;
  while (blo < bhi) {
    const int mid = (blo + bhi) >> 1;
    if (row_less(sb[h][mid], sn[h][mid], y)) blo = mid + 1; else bhi = mid;
  }
  const uint32_t r = atomicAdd(&a.bcnt[g * kMaxBuckets + blo], 1u);
  if (r >= (uint32_t)kMaxBucket) fail(a);
  atomicAdd(&a.bsum[g * kMaxBuckets + blo], a.ncount[X]);
  a.place[X] = ((uint32_t)blo << 24) | min(r, 0xFFFFFFu);
}

// Nodes of large groups moved to their buckets, every other node left where it is, into
// grouped2, with the bucket as the range the node is ordered within and the path count of
// the buckets before it.  Each workgroup scans the buckets of its (at most two) large
// groups for itself.
__global__ __launch_bounds__(kClassPer) void rscatter_kernel(TrieArgs a) {
  __shared__ uint32_t bs[2][kMaxBuckets + 1], bp[2][kMaxBuckets + 1];
  __shared__ uint32_t wsum[2][kMaxBuckets / 64];
  __shared__ uint32_t grp[2];
  __shared__ int oversized[2];
  const uint64_t nodes = node_count(a);
  const uint64_t lo = (uint64_t)blockIdx.x * kClassPer;
  if (lo >= nodes) return;
  if (threadIdx.x < 2) oversized[threadIdx.x] = 0;
  const uint64_t p = lo + threadIdx.x, ng = large_groups(a);
  uint32_t X = 0, g = 0xFFFFFFFFu;
  uint64_t u = 0;
  if (p < nodes) {
    X = a.grouped[p];
    u = a.unit[p];
    if ((uint32_t)u > (uint32_t)a.large) g = a.lgroup[a.nparent[X]];
    if ((uint64_t)g >= ng) g = 0xFFFFFFFFu;
  }
  const uint64_t last = min(lo + kClassPer, nodes) - 1;
  if (p == lo) grp[0] = g;
  if (p == last) grp[1] = g;
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int h = 0; h < 2; ++h) {
    const uint32_t gh = grp[h];
    if (gh == 0xFFFFFFFFu || (h == 1 && gh == grp[0])) continue;  // (uniform)
    const uint32_t c = threadIdx.x < kMaxBuckets ? a.bcnt[gh * kMaxBuckets + threadIdx.x] : 0u;
    if (c > (uint32_t)kMaxBucket) oversized[h] = 1;
    uint32_t x = c, z = threadIdx.x < kMaxBuckets ? a.bsum[gh * kMaxBuckets + threadIdx.x] : 0u;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64), v = __shfl_up(z, o, 64);
      if (lane >= o) { x += y; z += v; }
    }
    if (threadIdx.x < kMaxBuckets && lane == 63) { wsum[0][w] = x; wsum[1][w] = z; }
    __syncthreads();
    if (threadIdx.x < kMaxBuckets) {
      for (int q = 0; q < w; ++q) { x += wsum[0][q]; z += wsum[1][q]; }
      bs[h][threadIdx.x + 1] = x;
      bp[h][threadIdx.x + 1] = z;
      if (threadIdx.x == 0) { bs[h][0] = 0; bp[h][0] = 0; }
    }
    __syncthreads();
  }
  if (p >= nodes) return;
  if (g == 0xFFFFFFFFu) {
    a.grouped2[p] = X;
    a.unit2[p] = u;
    a.base2[p] = 0;
    return;
  }
  const int h = g == grp[0] ? 0 : 1;
  if (oversized[h]) {  // the call has failed (classify_kernel): nothing to order here
    a.grouped2[p] = X;
    a.unit2[p] = (p << 32) | 1;
    a.base2[p] = 0;
    return;
  }
  const uint32_t at = a.place[X], bk = at >> 24, g0 = (uint32_t)(u >> 32);
  const uint64_t dst = (uint64_t)g0 + bs[h][bk] + (at & 0xFFFFFFu);
  a.grouped2[dst] = X;
  a.unit2[dst] = ((uint64_t)(g0 + bs[h][bk]) << 32) | (bs[h][bk + 1] - bs[h][bk]);
  a.base2[dst] = bp[h][bk];
}

// What a node adds to the ranks of the paths through it: the paths through its earlier
// siblings and, if one ends there, the path that ends at its parent.  Every node adds up the
// path counts of the nodes of its range (a group, or a bucket of a large one, base: the
// buckets before it) with a smaller block; siblings' blocks are distinct.  A workgroup takes
// Threads / L consecutive positions, L lanes a node, and stages the blocks of the ranges
// they lie in, Threads rows at a time, in LDS: no sort, no barriers but around a stage, and
// any mixture of small and large ranges.  (Sorted by counting up to 64 siblings, by bitonic
// sorts up to 2,048 and in buckets, with the counts then gathered and scanned in sorted
// order: nine launches on two streams, about 120 us of a 1,048,576-event build; with the
// splitting four launches, 61 us, this one 22 us of them, 72 us for 405,319 nodes.)  The work
// grows with the ranges' sizes squared, up to a millisecond for 400,000 siblings, so a call that
// has failed already does none of it (400,000 one-frame paths, whose hashes collide, 2.19 ->
// 1.71 ms with the comparison sort that follows).
template <int L, int Threads>
__global__ __launch_bounds__(Threads) void order_kernel(TrieArgs a, const uint32_t *members, const uint64_t *unit,
                                                        const uint32_t *base) {
  constexpr int kPer = Threads / L;
  __shared__ uint64_t sb[Threads][kRowWords];
  __shared__ uint32_t sc[Threads];
  __shared__ uint8_t sn[Threads];
  __shared__ uint32_t first, end;
  const uint64_t nodes = node_count(a);
  if ((uint64_t)blockIdx.x * kPer >= nodes || a.ctr[kFail]) return;  // (after a failure no rank counts)
  const uint64_t p = (uint64_t)blockIdx.x * kPer + threadIdx.x / L;
  const int l = threadIdx.x % L;
  const bool in = p < nodes;
  if (threadIdx.x == 0) { first = 0xFFFFFFFFu; end = 0; }
  __syncthreads();
  uint32_t X = 0, s = 0, n = 0;
  if (in) {
    X = members[p];
    const uint64_t u = unit[p];
    s = (uint32_t)(u >> 32);
    n = (uint32_t)u;
    if (n > 1 && l == 0) {
      atomicMin(&first, s);
      atomicMax(&end, s + n);
    }
  }
  BlockRow y{};
  if (n > 1) node_row(a, X, y);
  __syncthreads();
  uint32_t sum = 0;
  const uint32_t r1 = (uint32_t)min((uint64_t)end, nodes);
  for (uint32_t t0 = first; t0 < r1; t0 += Threads) {  // (first is all ones when there is nothing to compare)
    const uint32_t m = min((uint32_t)Threads, r1 - t0);
    if (threadIdx.x < m) {
      const uint32_t Y = members[t0 + threadIdx.x];
      BlockRow r;
      node_row(a, Y, r);
      put_row(sb[threadIdx.x], &sn[threadIdx.x], r);
      sc[threadIdx.x] = a.ncount[Y];
    }
    __syncthreads();
    if (n > 1) {  // this stage's part of the node's range
      const uint32_t j0 = max(s, t0), j1 = min(s + n, t0 + m);
      for (uint32_t j = j0 + l; j < j1; j += L) sum += row_less(sb[j - t0], sn[j - t0], y) ? sc[j - t0] : 0u;
    }
    __syncthreads();
  }
#pragma unroll
  for (int o = L / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (l != 0 || !in) return;
  const uint32_t P = a.nparent[X];
  a.weight[X] = sum + (base ? base[p] : 0u) + (P == (uint32_t)a.nblocks ? (uint32_t)a.ctr[kTrieCtrEmpty] : a.nend[P]);
}

// A path's rank: the weights along its chain.  Eight lanes per path, which meet by three
// shuffles within the eight lanes.
constexpr int kRankLanes = 8;
__global__ __launch_bounds__(256) void rank_kernel(TrieArgs a) {
  const int64_t d = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kRankLanes;
  const int g = threadIdx.x % kRankLanes;
  const bool active = d < a.d;
  const uint32_t len = active ? a.plen[d] : 0u;
  const int64_t b0 = active ? a.pstart[d] / kBlk : 0, nb = (len + kBlk - 1) / kBlk;
  uint32_t part = 0;
  for (int64_t k = g; k < nb; k += kRankLanes) part += a.weight[a.occ[b0 + k]];
#pragma unroll
  for (int o = kRankLanes / 2; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
  if (!active || g != 0) return;
  if (part < (uint64_t)a.d) a.order[part] = (uint32_t)d;
  else fail(a);
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

void launch_trie_sort(const TrieArgs &args, int64_t d_old, hipStream_t s) {
  if (args.d <= 0) return;
  TrieArgs a = args;
  hipLaunchKernelGGL(clear_kernel, dim3(blocks_for((int64_t)a.cap, 256)), dim3(256), 0, s, a);
  if (d_old > 0) hipLaunchKernelGGL(fill_kernel, dim3(blocks_for(d_old, 256)), dim3(256), 0, s, a, d_old);
  if (a.nblocks > 0) {
    const unsigned per256 = blocks_for(a.nblocks, 256);
    hipLaunchKernelGGL(insert_kernel, dim3(per256), dim3(256), 0, s, a);
    hipLaunchKernelGGL(resolve_kernel, dim3(per256), dim3(256), 0, s, a);
    const int64_t link_grid = std::max<int64_t>(1, std::min<int64_t>(blocks_for(a.nblocks, 1024), 512));
    hipLaunchKernelGGL(link_kernel, dim3((unsigned)link_grid), dim3(kLinkThreads), 0, s, a);
    // in a small trie counting within whole groups is cheaper than three more launches: a
    // wave to a node, which spreads 2,048 nodes over 256 workgroups (1,877 nodes in one
    // group: 19 us; 69 us with sixteen lanes to a node, in 30 workgroups)
    const bool small = a.nblocks <= kSmallTrie;
    a.large = small ? (int32_t)kSmallTrie : kLarge;
    hipLaunchKernelGGL(alloc_kernel, dim3(blocks_for(a.nblocks + 1, kAllocThreads * kAllocPer)), dim3(kAllocThreads),
                       0, s, a);
    hipLaunchKernelGGL(scatter_kernel, dim3(per256), dim3(256), 0, s, a);
    if (small) {
      hipLaunchKernelGGL((order_kernel<64, 512>), dim3(blocks_for(a.nblocks, 512 / 64)), dim3(512), 0, s, a,
                         a.grouped, a.unit, (const uint32_t *)nullptr);
    } else {
      const unsigned large = (unsigned)std::min<int64_t>(a.large_cap, 256);
      hipLaunchKernelGGL(split_kernel, dim3(kSamples / kSplitPer, large), dim3(kSplitThreads), 0, s, a);
      hipLaunchKernelGGL(classify_kernel, dim3(blocks_for(a.nblocks, kClassPer)), dim3(kClassPer), 0, s, a);
      hipLaunchKernelGGL(rscatter_kernel, dim3(blocks_for(a.nblocks, kClassPer)), dim3(kClassPer), 0, s, a);
      hipLaunchKernelGGL((order_kernel<4, 512>), dim3(blocks_for(a.nblocks, 512 / 4)), dim3(512), 0, s, a,
                         a.grouped2, a.unit2, a.base2);
    }
  }
  hipLaunchKernelGGL(rank_kernel, dim3(blocks_for(a.d * kRankLanes, 256)), dim3(256), 0, s, a);
}

}  // namespace cct
