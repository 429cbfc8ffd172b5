// Bottom-up view of the tree: the metrics of every frame aggregated over all the call
// paths it appears on.  The flame-graph view of the paper offers a top-down view (the
// tree itself) and a bottom-up view that aggregates the metrics of the same node across
// different call paths (Implementation, "GUI", "Flame Graph Visualization").
//
// For a frame f:
//   excl(f) = sum over the nodes labelled f of their exclusive sums (the events whose
//             path ends with f);
//   incl(f) = sum over the events whose path contains f, each counted once however often
//             f recurs on its path = sum of the inclusive sums of the topmost nodes
//             labelled f (no proper ancestor labelled f): every such event passes through
//             exactly one of them.
//
// On the canonical tree (preorder ids, subtree of u = ids [u, subend[u])):
//   1. the nodes 1 .. U-1 are sorted by frame with a stable radix sort (one pass for each
//      of the four bytes in which the frames differ), so each frame's nodes form a group in
//      preorder;
//   2. a node is topmost iff no earlier node of its group has a subtree that reaches past
//      it: one exclusive max-scan over (group index << 32 | subend) decides every node
//      (an earlier group has a smaller high word);
//   3. the nodes' exclusive sums and the topmost nodes' inclusive sums are gathered in
//      sorted order and summed per group: a group is a run of the sorted nodes, so a tile
//      of 1,024 nodes meets at most as many groups, sums them in LDS and stores all but
//      its first and last, which may go on in other tiles.
//
// For 2.09 million nodes of 171,461 frames (2 metrics) the kernels took 515 us when every node
// first learnt its group in node order and the ingest's aggregation kernels summed them
// (57 us for the scattered groups, 190 us for the two aggregations), the sort's four
// passes ran from 2,048-element tiles (185 us); 278 us now, of which the four sort passes 100 us,
// the tags 34 us and the sums 82 us.
#include <algorithm>

#include "common.h"

namespace cct {

namespace {

// ---- stable LSD radix sort of (uint32 key, uint32 value) pairs ---------------------------
// A tile is 8 waves of 512 consecutive elements.  4,096 elements on 256 digits leave runs
// of 16 keys (64 bytes) per digit in the output; they are put in order in LDS first, so
// that a run is stored by neighbouring lanes (43 us a pass of 2.1 million pairs with
// 2,048 a tile and every element stored from where it was read, 15 - 17 us so).
constexpr int kRsThreads = 512, kRsPerThread = 8, kRsTile = kRsThreads * kRsPerThread;
constexpr int kRsWaves = kRsThreads / 64;

// digit histogram of one tile, stored digit-major: hist[digit * nblk + block].  The first
// pass also leaves the bits in which the tile's keys differ from the first key (the host
// leaves out the passes over digits that never differ) and the time at which it began.
template <bool First>
__global__ __launch_bounds__(kRsThreads) void rs_hist_kernel(const uint32_t *keys, int64_t n, int shift, int64_t nblk,
                                                            uint64_t *hist, unsigned long long *bits) {
  __shared__ uint32_t h[256], differ;
  const int tid = threadIdx.x;
  if (First && blockIdx.x == 0 && tid == 0) bits[nblk] = (unsigned long long)wall_clock64();
  if (tid < 256) h[tid] = 0;
  if (tid == 0) differ = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)blockIdx.x * kRsTile + tid;
  uint32_t key[kRsPerThread];
#pragma unroll
  for (int k = 0; k < kRsPerThread; ++k) {
    const int64_t i = t0 + (int64_t)k * kRsThreads;
    key[k] = i < n ? keys[i] : 0u;
  }
#pragma unroll
  for (int k = 0; k < kRsPerThread; ++k)
    if (t0 + (int64_t)k * kRsThreads < n) atomicAdd(&h[(key[k] >> shift) & 255u], 1u);
  if (First) {
    const uint32_t k0 = keys[0];
    uint32_t d = 0;
#pragma unroll
    for (int k = 0; k < kRsPerThread; ++k)
      if (t0 + (int64_t)k * kRsThreads < n) d |= key[k] ^ k0;
    for (int o = 32; o > 0; o >>= 1) d |= __shfl_xor(d, o, 64);
    if ((tid & 63) == 0 && d) atomicOr(&differ, d);
  }
  __syncthreads();
  if (tid < 256) hist[(int64_t)tid * nblk + blockIdx.x] = h[tid];
  if (First && tid == 0) bits[blockIdx.x] = differ;
}

// the bits in which any two keys differ, and the time of the first pass, to the host
__global__ __launch_bounds__(1024) void rs_bits_kernel(const unsigned long long *bits, int64_t nblk,
                                                       unsigned long long *host) {
  __shared__ uint32_t differ;
  if (threadIdx.x == 0) differ = 0;
  __syncthreads();
  uint32_t d = 0;
  for (int64_t b = threadIdx.x; b < nblk; b += 1024) d |= (uint32_t)bits[b];
  for (int o = 32; o > 0; o >>= 1) d |= __shfl_xor(d, o, 64);
  if ((threadIdx.x & 63) == 0 && d) atomicOr(&differ, d);
  __syncthreads();
  if (threadIdx.x == 0) {
    host[0] = differ;
    host[1] = bits[nblk];
  }
}

// Scatter of one tile to its digits' places (offs: exclusive scan of the digit-major
// histogram).  A wave reads its 512 elements in rounds of 64: 8 ballots find the lanes
// with the same digit, and the wave's own counts the rounds before, so equal keys keep
// their order and the rounds need no barrier.  The first pass takes vals == nullptr for
// the sequence 1, 2, ...
__global__ __launch_bounds__(kRsThreads) void rs_scatter_kernel(const uint32_t *keys, const uint32_t *vals, int64_t n,
                                                               int shift, int64_t nblk, const uint64_t *offs,
                                                               uint32_t *keys_out, uint32_t *vals_out) {
  __shared__ uint32_t cnt[kRsWaves][256];       // a wave's elements of a digit; then the place of its first
  __shared__ uint32_t base[256], wsum[4];       // output position - place in the tile, per digit
  __shared__ uint32_t skey[kRsTile], sval[kRsTile];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t t0 = (int64_t)blockIdx.x * kRsTile, w0 = t0 + wave * (64 * kRsPerThread) + lane;
  uint32_t key[kRsPerThread], val[kRsPerThread], rank[kRsPerThread];
#pragma unroll
  for (int k = 0; k < kRsPerThread; ++k) {
    const int64_t i = w0 + k * 64;
    key[k] = i < n ? keys[i] : 0u;
    val[k] = i < n ? (vals ? vals[i] : (uint32_t)(i + 1)) : 0u;
  }
  uint32_t off = 0;
  if (tid < 256) off = (uint32_t)offs[(int64_t)tid * nblk + blockIdx.x];
  for (int c = lane; c < 256; c += 64) cnt[wave][c] = 0;
  __syncthreads();
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  volatile uint32_t *mine = cnt[wave];
#pragma unroll
  for (int k = 0; k < kRsPerThread; ++k) {
    const bool valid = w0 + k * 64 < n;
    const uint32_t d = (key[k] >> shift) & 255u;
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint64_t ones = __ballot((d >> b) & 1u);
      same &= ((d >> b) & 1u) ? ones : ~ones;
    }
    const uint32_t before = valid ? mine[d] : 0u, in_round = (uint32_t)__popcll(same & below);
    rank[k] = before + in_round;
    __builtin_amdgcn_wave_barrier();
    if (valid && in_round == 0) mine[d] = before + (uint32_t)__popcll(same);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  uint32_t total = 0, incl = 0;
  if (tid < 256) {  // one digit a thread: the waves' counts and the digits' totals become places
#pragma unroll
    for (int w = 0; w < kRsWaves; ++w) {
      const uint32_t c = cnt[w][tid];
      cnt[w][tid] = total;
      total += c;
    }
    incl = total;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
  }
  __syncthreads();
  if (tid < 256) {
    uint32_t first = incl - total;
    for (int w = 0; w < wave; ++w) first += wsum[w];
    base[tid] = off - first;  // (mod 2^32)
#pragma unroll
    for (int w = 0; w < kRsWaves; ++w) cnt[w][tid] += first;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRsPerThread; ++k)
    if (w0 + k * 64 < n) {
      const uint32_t at = cnt[wave][(key[k] >> shift) & 255u] + rank[k];
      skey[at] = key[k];
      sval[at] = val[k];
    }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRsPerThread; ++k) {
    const int j = k * kRsThreads + tid;
    if (t0 + j < n) {
      const uint32_t kk = skey[j];
      const uint32_t pos = base[(kk >> shift) & 255u] + (uint32_t)j;
      keys_out[pos] = kk;
      vals_out[pos] = sval[j];
    }
  }
}

// ---- exclusive max-scan of uint64 (identity 0) -------------------------------------------
constexpr int kMsThreads = 256, kMsPer = 4, kMsRows = kMsThreads * kMsPer;

__device__ inline uint64_t umax64(uint64_t a, uint64_t b) { return a > b ? a : b; }
__device__ inline uint64_t xor_u64(uint64_t v, int o) {
  const uint32_t lo = __shfl_xor((uint32_t)v, o, 64), hi = __shfl_xor((uint32_t)(v >> 32), o, 64);
  return ((uint64_t)hi << 32) | lo;
}
__device__ inline uint64_t up_u64(uint64_t v, int o) {
  const uint32_t lo = __shfl_up((uint32_t)v, o, 64), hi = __shfl_up((uint32_t)(v >> 32), o, 64);
  return ((uint64_t)hi << 32) | lo;
}

// exclusive max-scan of the block maxima in place (one workgroup)
__global__ __launch_bounds__(kMsThreads) void ms_blocks_kernel(uint64_t *blk, int64_t nblk) {
  __shared__ uint64_t part[kMsThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint64_t carry = 0;
  for (int64_t b0 = 0; b0 < nblk; b0 += kMsThreads) {
    const int64_t b = b0 + tid;
    const uint64_t v = b < nblk ? blk[b] : 0;
    uint64_t x = v;  // inclusive within the wave
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t y = up_u64(x, o);
      if (lane >= o) x = umax64(x, y);
    }
    if (lane == 63) part[wave] = x;
    __syncthreads();
    uint64_t before = carry;
    for (int w = 0; w < wave; ++w) before = umax64(before, part[w]);
    const uint64_t prev = up_u64(x, 1);  // every lane takes part in the shuffle
    const uint64_t excl = lane ? umax64(before, prev) : before;
    uint64_t tot = carry;
    for (int w = 0; w < kMsThreads / 64; ++w) tot = umax64(tot, part[w]);
    __syncthreads();
    if (b < nblk) blk[b] = excl;
    carry = tot;
  }
}

// ---- the view -----------------------------------------------------------------------------
// Tiles of kMsRows sorted nodes; thread t has rows 4t .. 4t+3 of its tile.

// the group heads of every tile counted
__global__ __launch_bounds__(kMsThreads) void bu_heads_kernel(const uint32_t *K, int64_t n, uint64_t *heads) {
  __shared__ uint32_t part[kMsThreads / 64];
  const int64_t r0 = (int64_t)blockIdx.x * kMsRows + threadIdx.x;
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < kMsPer; ++k) {
    const int64_t i = r0 + (int64_t)k * kMsThreads;
    c += (uint32_t)__popcll(__ballot(i < n && (i == 0 || K[i] != K[i - 1])));
  }
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kMsThreads / 64; ++w) c += part[w];
    heads[blockIdx.x] = c;
  }
}

// tag of sorted position i: (group << 32) | subend of its node, and every tile's largest;
// first: exclusive scan of the tiles' heads
__global__ __launch_bounds__(kMsThreads) void bu_tag_kernel(const uint32_t *K, const uint32_t *V, const uint64_t *first,
                                                           const uint32_t *subend, int64_t n, uint64_t *tag,
                                                           uint64_t *blk) {
  __shared__ uint32_t part[kMsThreads / 64];
  __shared__ uint64_t pmax[kMsThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kMsRows + (int64_t)tid * kMsPer;
  uint32_t end[kMsPer], count[kMsPer], c = 0;
  uint32_t prev = r0 > 0 && r0 < n ? K[r0 - 1] : 0u;
#pragma unroll
  for (int k = 0; k < kMsPer; ++k) {
    const int64_t i = r0 + k;
    end[k] = i < n ? subend[V[i]] : 0u;
    const uint32_t key = i < n ? K[i] : prev;
    c += i < n && (i == 0 || key != prev);
    count[k] = c;
    prev = key;
  }
  uint32_t x = c;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) part[wave] = x;
  __syncthreads();
  uint64_t g = first[blockIdx.x] + x - c;
  for (int w = 0; w < wave; ++w) g += part[w];
  uint64_t m = 0;
#pragma unroll
  for (int k = 0; k < kMsPer; ++k)
    if (r0 + k < n) {
      const uint64_t v = ((g + count[k] - 1) << 32) | end[k];
      tag[r0 + k] = v;
      m = umax64(m, v);
    }
  for (int o = 32; o > 0; o >>= 1) m = umax64(m, xor_u64(m, o));
  if (lane == 0) pmax[wave] = m;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kMsThreads / 64; ++w) m = umax64(m, pmax[w]);
    blk[blockIdx.x] = m;
  }
}

__global__ void bu_clear_kernel(uint64_t *ex, uint64_t *in, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) ex[i] = in[i] = 0;
}

// Frames and sums of the groups.  blk: exclusive max-scan of the tiles' largest tags; ex
// and in are zero.  The rows of the sums come from anywhere in the tree (an L2 line a
// node and array); 32 KB of LDS hold two metrics of a tile's groups, so more metrics take
// further turns and four workgroups (32,800 bytes each) still share a CU.
template <int M>
__global__ __launch_bounds__(kMsThreads) void bu_sums_kernel(const uint32_t *K, const uint32_t *V, const uint64_t *tag,
                                                            const uint64_t *blk, const uint64_t *excl,
                                                            const uint64_t *incl, int64_t n, uint32_t *frames,
                                                            unsigned long long *ex, unsigned long long *in) {
  constexpr int C = M < 2 ? 1 : 2;
  __shared__ unsigned long long acc[kMsRows * 2 * C];  // [group][exclusive C, inclusive C]
  __shared__ uint64_t part[kMsThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t t0 = (int64_t)blockIdx.x * kMsRows, r0 = t0 + (int64_t)tid * kMsPer;
  const uint64_t g0 = tag[t0] >> 32;
  const int groups = (int)((tag[min(t0 + kMsRows, n) - 1] >> 32) - g0) + 1;
  // topmost nodes: what the earlier rows' tags reach
  uint64_t v[kMsPer], m = 0;
  uint32_t node[kMsPer];
#pragma unroll
  for (int k = 0; k < kMsPer; ++k) {
    v[k] = r0 + k < n ? tag[r0 + k] : 0;
    node[k] = r0 + k < n ? V[r0 + k] : 0u;
    m = umax64(m, v[k]);
  }
  uint64_t x = m;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = up_u64(x, o);
    if (lane >= o) x = umax64(x, y);
  }
  if (lane == 63) part[wave] = x;
  __syncthreads();
  uint64_t run = blk[blockIdx.x];
  for (int w = 0; w < wave; ++w) run = umax64(run, part[w]);
  const uint64_t prev = up_u64(x, 1);  // every lane takes part in the shuffle
  if (lane) run = umax64(run, prev);
  bool top[kMsPer];
  uint64_t pg = r0 > 0 && r0 < n ? tag[r0 - 1] >> 32 : ~0ull;
#pragma unroll
  for (int k = 0; k < kMsPer; ++k) {
    const uint64_t g = v[k] >> 32;
    top[k] = (run >> 32) != g || (uint64_t)node[k] >= (run & 0xFFFFFFFFull);
    run = umax64(run, v[k]);
    if (r0 + k < n && g != pg) frames[g] = K[r0 + k];
    pg = g;
  }
  // (row 0 of a tree's first group: nothing before it, run == 0, and the group is 0 as
  // well; a node is at least 1, so it counts as topmost all the same)
#pragma unroll
  for (int c0 = 0; c0 < M; c0 += C) {
    constexpr int W = 2 * C;
    const int cn = M - c0 < C ? M - c0 : C;
    uint64_t e[kMsPer][C], q[kMsPer][C];
#pragma unroll
    for (int k = 0; k < kMsPer; ++k)
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const bool ok = r0 + k < n && j < cn;
        e[k][j] = ok ? excl[(int64_t)node[k] * M + c0 + j] : 0;
        q[k][j] = ok && top[k] ? incl[(int64_t)node[k] * M + c0 + j] : 0;
      }
    for (int i = tid; i < groups * W; i += kMsThreads) acc[i] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kMsPer; ++k) {
      const bool last = k == kMsPer - 1 || r0 + k + 1 >= n || (v[k + 1 < kMsPer ? k + 1 : k] >> 32) != (v[k] >> 32);
      if (last) {
        if (r0 + k < n) {
          unsigned long long *at = acc + (uint32_t)((v[k] >> 32) - g0) * W;
#pragma unroll
          for (int j = 0; j < C; ++j) {
            if (e[k][j]) atomicAdd(at + j, (unsigned long long)e[k][j]);
            if (q[k][j]) atomicAdd(at + C + j, (unsigned long long)q[k][j]);
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < C; ++j) {
          e[k + 1 < kMsPer ? k + 1 : k][j] += e[k][j];
          q[k + 1 < kMsPer ? k + 1 : k][j] += q[k][j];
        }
      }
    }
    __syncthreads();
    for (int i = tid; i < groups * W; i += kMsThreads) {
      const int g = i / W, j = i % W % C;
      if (j >= cn) continue;
      unsigned long long *out = (i % W < C ? ex : in) + (int64_t)(g0 + g) * M + c0 + j;
      if (g == 0 || g == groups - 1) {
        if (acc[i]) atomicAdd(out, acc[i]);
      } else {
        *out = acc[i];
      }
    }
    __syncthreads();
  }
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

int64_t radix_blocks(int64_t n) { return (n + kRsTile - 1) / kRsTile; }
int64_t bu_tiles(int64_t n) { return (n + kMsRows - 1) / kMsRows; }

void launch_radix_pass(const uint32_t *keys, const uint32_t *vals, int64_t n, int shift, uint64_t *hist, uint64_t *offs,
                       uint64_t *scan_blk, uint32_t *keys_out, uint32_t *vals_out, hipStream_t s) {
  const int64_t nblk = radix_blocks(n);
  hipLaunchKernelGGL(rs_hist_kernel<false>, dim3((unsigned)nblk), dim3(kRsThreads), 0, s, keys, n, shift, nblk, hist,
                     (unsigned long long *)nullptr);
  launch_scan(hist, 256 * nblk, 1, scan_blk, offs, s);
  hipLaunchKernelGGL(rs_scatter_kernel, dim3((unsigned)nblk), dim3(kRsThreads), 0, s, keys, vals, n, shift, nblk, offs,
                     keys_out, vals_out);
}
void launch_radix_bits(const uint32_t *keys, int64_t n, uint64_t *hist, unsigned long long *bits,
                       unsigned long long *host, hipStream_t s) {
  const int64_t nblk = radix_blocks(n);
  hipLaunchKernelGGL(rs_hist_kernel<true>, dim3((unsigned)nblk), dim3(kRsThreads), 0, s, keys, n, 0, nblk, hist, bits);
  hipLaunchKernelGGL(rs_bits_kernel, dim3(1), dim3(1024), 0, s, bits, nblk, host);
}
void launch_radix_first(const uint32_t *keys, int64_t n, const uint64_t *hist, uint64_t *offs, uint64_t *scan_blk,
                        uint32_t *keys_out, uint32_t *vals_out, hipStream_t s) {
  const int64_t nblk = radix_blocks(n);
  launch_scan(hist, 256 * nblk, 1, scan_blk, offs, s);
  hipLaunchKernelGGL(rs_scatter_kernel, dim3((unsigned)nblk), dim3(kRsThreads), 0, s, keys, (const uint32_t *)nullptr, n,
                     0, nblk, offs, keys_out, vals_out);
}

void launch_bu_heads(const uint32_t *K, int64_t n, uint64_t *heads, hipStream_t s) {
  hipLaunchKernelGGL(bu_heads_kernel, dim3((unsigned)bu_tiles(n)), dim3(kMsThreads), 0, s, K, n, heads);
}
void launch_bu_tag(const uint32_t *K, const uint32_t *V, const uint64_t *first, const uint32_t *subend, int64_t n,
                   uint64_t *tag, uint64_t *blk, hipStream_t s) {
  const int64_t nt = bu_tiles(n);
  hipLaunchKernelGGL(bu_tag_kernel, dim3((unsigned)nt), dim3(kMsThreads), 0, s, K, V, first, subend, n, tag, blk);
  hipLaunchKernelGGL(ms_blocks_kernel, dim3(1), dim3(kMsThreads), 0, s, blk, nt);
}
void launch_bu_sums(const uint32_t *K, const uint32_t *V, const uint64_t *tag, const uint64_t *blk, const uint64_t *excl,
                    const uint64_t *incl, int64_t n, int64_t G, int32_t m, uint32_t *frames, uint64_t *ex, uint64_t *in,
                    hipStream_t s) {
  hipLaunchKernelGGL(bu_clear_kernel, dim3(std::min(blocks_for(G * m, 256), 2048u)), dim3(256), 0, s, ex, in, G * m);
  switch (m) {
#define CCT_CASE(M)                                                                                              \
  case M:                                                                                                        \
    hipLaunchKernelGGL(bu_sums_kernel<M>, dim3((unsigned)bu_tiles(n)), dim3(kMsThreads), 0, s, K, V, tag, blk,   \
                       excl, incl, n, frames, (unsigned long long *)ex, (unsigned long long *)in);               \
    break;
    CCT_CASE(1) CCT_CASE(2) CCT_CASE(3) CCT_CASE(4) CCT_CASE(5) CCT_CASE(6) CCT_CASE(7) CCT_CASE(8)
#undef CCT_CASE
  }
}

}  // namespace cct
