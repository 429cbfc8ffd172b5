// Analysis queries as data-parallel filters over the tree.  The paper's example analyses
// walk the tree and flag nodes whose metric ratio crosses a threshold: a kernel whose
// time is a large share of the root's (hotspot), a frame whose GPU time per kernel is
// small (kernel fusion), a frame whose CPU time is large against its GPU time (CPU
// latency) (Implementation, "Performance Analyzer", "Example Analyses").
//
// One predicate covers them: node v matches when a(v) / b(v) is above (or below) the
// threshold p / q, tested without division as a(v) * q > p * b(v) (or <) in exact 128-bit
// integer arithmetic; a(v) is one of the node's sums, b(v) is 1, another of the node's
// sums, or the root's inclusive sum.  Optionally only leaves (nodes without children)
// match.
//
// Two passes over tiles of kFilterTile nodes list the matches in ascending id order
// (preorder): the first evaluates the predicate once per node and keeps it as one bit
// (a wave's ballot is the mask word of its 64 nodes) plus a match count per tile; the second
// pass reads only the mask and writes each match's id at its tile's offset plus its rank
// among the tile's earlier matches.  A workgroup of the second pass adds up the counts of
// the tiles before its own (a few thousand for millions of nodes), and the last one hands
// the number of matches to the host.
#include <mutex>

#include "common.h"

namespace cct {

namespace {

constexpr int kFilterThreads = 256;
constexpr int kFilterRounds = kFilterTile / kFilterThreads;  // nodes per thread in the first pass
constexpr int kTileWords = kFilterTile / 64;                 // mask words per tile
constexpr int kScanThreads = 1024, kScanPer = 4;             // tile-count scan: one workgroup
static_assert(kFilterTile % kFilterThreads == 0 && kTileWords <= 64, "tile shape");

// a * q versus p * b over unsigned 128-bit products: -1, 0, +1
__device__ inline int cmp_products(uint64_t a, uint64_t q, uint64_t p, uint64_t b) {
  const uint64_t lo1 = a * q, hi1 = __umul64hi(a, q);
  const uint64_t lo2 = p * b, hi2 = __umul64hi(p, b);
  if (hi1 != hi2) return hi1 < hi2 ? -1 : 1;
  if (lo1 != lo2) return lo1 < lo2 ? -1 : 1;
  return 0;
}

__device__ inline bool node_matches(const FilterArgs &a, int64_t v) {
  const uint64_t *num = a.num_excl ? a.excl : a.incl;
  const uint64_t x = num[v * a.m + a.num_metric];
  uint64_t y = 1;
  if (a.den_kind == kDenMetric) y = (a.den_excl ? a.excl : a.incl)[v * a.m + a.den_metric];
  else if (a.den_kind == kDenRoot) y = a.incl[a.den_metric];
  const int c = cmp_products(x, a.thr_den, a.thr_num, y);
  const bool hit = a.op > 0 ? c > 0 : c < 0;
  return hit && (!a.leaves_only || a.subend[v] == (uint32_t)(v + 1));  // a leaf's subtree is itself
}

// mask[w] bit l: node 64 w + l matches (every word of every tile is written, zero past U);
// count[t]: matches in tile t
__global__ __launch_bounds__(kFilterThreads) void filter_mask_kernel(FilterArgs a, uint64_t *mask, uint32_t *count,
                                                                     unsigned long long *started) {
  if (started) stamp(started);
  __shared__ uint32_t wave_count[kFilterThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kFilterTile;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bool hit[kFilterRounds];
#pragma unroll
  for (int r = 0; r < kFilterRounds; ++r) {
    const int64_t v = base + r * kFilterThreads + threadIdx.x;
    hit[r] = v < a.u && node_matches(a, v);
  }
  uint32_t c = 0;
#pragma unroll
  for (int r = 0; r < kFilterRounds; ++r) {
    const uint64_t bits = __ballot(hit[r]);
    c += (uint32_t)__popcll(bits);
    if (lane == 0) mask[(base + r * kFilterThreads + wave * 64) >> 6] = bits;
  }
  if (lane == 0) wave_count[wave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < kFilterThreads / 64; ++w) t += wave_count[w];
    count[blockIdx.x] = t;
  }
}

// pos[t] = count[0] + ... + count[t - 1] for t <= T (pos[T]: all matches), for trees of more
// than kFilterDirect tiles; a single workgroup walks the counts kScanThreads * kScanPer at a time.
// (Without it every workgroup of the second pass adds up the earlier tiles' counts, which come from
// the caches but grow with the square of the tiles: calls with and without the scan took 43 and
// 43 us at 2,900 tiles, 65 and 66 at 8,800, 98 and 95 at 17,600, 143 and 136 at 29,300.  The
// line only bounds the square.)
__global__ __launch_bounds__(kScanThreads) void filter_scan_kernel(const uint32_t *count, int64_t T, uint64_t *pos) {
  __shared__ uint32_t wave_sum[kScanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint64_t carry = 0;
  for (int64_t t0 = 0; t0 < T; t0 += kScanThreads * kScanPer) {
    const int64_t t = t0 + (int64_t)tid * kScanPer;
    uint32_t c[kScanPer], mine = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      c[k] = t + k < T ? count[t + k] : 0;
      mine += c[k];
    }
    uint32_t x = mine;  // inclusive scan over the wave
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    if (lane == 63) wave_sum[wave] = x;
    __syncthreads();
    uint32_t before = 0, total = 0;  // at most kFilterTile * kScanThreads * kScanPer < 2^32
    for (int w = 0; w < kScanThreads / 64; ++w) {
      const uint32_t v = wave_sum[w];
      before += w < wave ? v : 0;
      total += v;
    }
    uint64_t run = carry + before + (x - mine);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      if (t + k < T) pos[t + k] = run;
      run += c[k];
    }
    carry += total;
    __syncthreads();  // wave_sum is rewritten by the next round
  }
  if (tid == 0) pos[T] = carry;
}

// One wave per tile, kFilterWaves tiles per workgroup.  pos null: the workgroup adds up the
// counts of the tiles before its own.  Lanes below kTileWords hold the tile's mask words and
// an inclusive scan of their bit counts; then word by word, each set bit's lane writes its
// node id.  The last tile's wave writes the number of matches and, if asked, the time once its own
// ids are written: its workgroup is dispatched last (4,222,948 nodes: 18.0 us for 67 matches, 18.7
// for 3,967,503; 16.2 and 16.3 if it is read before the ids; 20.0 and 21.4 with the launch of a
// kernel after this one, which made the call 1.7 us longer).  (With
// the scan as a launch between the passes, a copy of the count, two timing events and a
// blocking wait, a call over 4,222,948 nodes took 47 us, 40 us so, 13 of them the mask.)
constexpr int64_t kFilterDirect = 8192;
constexpr int kFilterWaves = 4;
__global__ __launch_bounds__(64 * kFilterWaves) void filter_write_kernel(const uint64_t *mask, const uint32_t *count,
                                                                         int64_t T, const uint64_t *pos,
                                                                         int64_t capacity, int64_t *out,
                                                                         unsigned long long *total,
                                                                         unsigned long long *ended) {
  __shared__ uint32_t part[kFilterWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t first = (int64_t)blockIdx.x * kFilterWaves, tile = first + wave;
  const uint64_t mine = tile < T && lane < kTileWords ? mask[tile * kTileWords + lane] : 0;
  int64_t base = 0;
  if (pos) {
    base = tile < T ? (int64_t)pos[tile] : 0;
  } else {  // (fewer than 2^32 nodes, so the sums fit 32 bits)
    uint32_t x = 0;
    for (int64_t t = threadIdx.x; t < first; t += 64 * kFilterWaves) x += count[t];
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if (lane == 0) part[wave] = x;
    __syncthreads();
    for (int w = 0; w < kFilterWaves; ++w) base += part[w];
    for (int64_t t = first; t < tile && t < T; ++t) base += count[t];
  }
  if (tile >= T) return;
  int incl = __popcll(mine);
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(incl, d);
    if (lane >= d) incl += t;
  }
  if (tile == T - 1 && lane == kTileWords - 1) *total = (unsigned long long)base + (unsigned long long)incl;
  const uint64_t below = (1ull << lane) - 1;
  for (int j = 0; j < kTileWords && base < capacity; ++j) {
    const uint32_t lo = __shfl((uint32_t)mine, j), hi = __shfl((uint32_t)(mine >> 32), j);
    const uint64_t word = ((uint64_t)hi << 32) | lo;
    const int before = __shfl(incl, j) - __popcll(word);  // matches of the tile's earlier words
    if ((word >> lane) & 1) {
      const int64_t k = base + before + __popcll(word & below);
      if (k < capacity) __builtin_nontemporal_store(tile * kFilterTile + j * 64 + lane, &out[k]);
    }
  }
  if (ended && tile == T - 1) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0) *ended = (unsigned long long)wall_clock64();
  }
}

// Scratch of the filter entry point that allocates nothing: the mask words, tile counts
// and tile offsets of up to kFilterStaticTiles tiles, laid out as filter_static_layout
// says.  Each GPU holds its own copy for the life of the process; every call on a GPU
// reuses it, so calls that overlap on one GPU race.  Host code never uses this name as an
// address (on the host it only stands for the symbol): the device address comes from
// hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[kFilterStaticBytes];

}  // namespace

int64_t filter_tiles(int64_t u) { return (u + kFilterTile - 1) / kFilterTile; }

FilterScratch filter_static_layout(void *base) {
  unsigned char *b = static_cast<unsigned char *>(base);
  FilterScratch f;
  f.mask = reinterpret_cast<uint64_t *>(b);
  f.count = reinterpret_cast<uint32_t *>(b + kFilterStaticTiles * kTileWords * 8);
  f.pos = reinterpret_cast<uint64_t *>(b + kFilterStaticTiles * (kTileWords * 8 + 4));
  return f;
}
static_assert(kFilterStaticTiles * (kTileWords * 8 + 4 + 8) + 8 <= kFilterStaticBytes, "static filter scratch");
static_assert((kFilterStaticTiles * (kTileWords * 8 + 4)) % 8 == 0, "pos alignment");

void *filter_static_scratch() {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void *ptr[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    ptr[dev] = p;
  }
  return ptr[dev];
}

void launch_filter(const FilterArgs &a, const FilterScratch &f, int64_t capacity, int64_t *out,
                   unsigned long long *total, unsigned long long *times, hipStream_t s) {
  const int64_t T = filter_tiles(a.u);  // (at least one: the root)
  hipLaunchKernelGGL(filter_mask_kernel, dim3((unsigned)T), dim3(kFilterThreads), 0, s, a, f.mask, f.count, times);
  const uint64_t *pos = nullptr;
  if (T > kFilterDirect) {
    hipLaunchKernelGGL(filter_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, f.count, T, f.pos);
    pos = f.pos;
  }
  hipLaunchKernelGGL(filter_write_kernel, dim3((unsigned)((T + kFilterWaves - 1) / kFilterWaves)),
                     dim3(64 * kFilterWaves), 0, s, f.mask, f.count, T, pos, capacity, out, total,
                     times ? times + 1 : nullptr);
}

}  // namespace cct
