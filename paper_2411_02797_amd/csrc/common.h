// Internal definitions shared by the HIP kernels and the host runtime of libcct.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cct {

// ---- unique-path table -------------------------------------------------------
// One 16-byte entry per slot.  word = (tag << 32) | ref, where ref is a path id of the
// tree's path store, or kEventRef | event index for a path first seen in the current
// call; it is claimed with one 64-bit CAS.  info tells where the slot's frames live and
// how many there are, so a lookup needs one memory round trip: written by the claimer
// right after its CAS (readers that still see kEmptyInfo fall back to ref).
struct Slot {
  uint64_t word;
  uint64_t info;
};
constexpr uint64_t kEmptySlot = ~0ull;
constexpr uint64_t kEmptyInfo = ~0ull;
constexpr uint32_t kEventRef = 0x80000000u;
constexpr uint32_t kRefMask = 0x7FFFFFFFu;
// info = (first frame << 24) | (in path store << 23) | length; lengths >= kInfoLongLen
// are stored as kInfoLongLen (their exact length is then read through ref).
constexpr uint64_t kInfoLongLen = 0x7FFFFF;
__host__ __device__ inline uint64_t make_info(uint64_t base, bool store, uint64_t len) {
  return (base << 24) | ((uint64_t)store << 23) | (len < kInfoLongLen ? len : kInfoLongLen);
}

// ---- ingest tiling -------------------------------------------------------------
constexpr int kIngestThreads = 1024;    // 16 waves of 64 (4 per SIMD), each with its own tile loop
constexpr int kWaveEvents = 63;         // max events per wave tile (lane j holds offset j, j <= 63)
constexpr int kLaneBlocks = 2;          // 16-frame blocks held by each lane of a wave tile
constexpr int kWaveFrames = 64 * 16 * kLaneBlocks;  // frames of a wave tile
constexpr int kCacheEntries = 4096;     // LDS resolved-path cache entries per workgroup

// ---- counters written by the ingest kernels --------------------------------------
enum Counter { kCtrNew = 0, kCtrError = 2, kCtrOverflow = 3, kCtrNewLen = 4,
               kCtrCount = 8 };
enum ErrorBits { kErrOffsets = 1 };
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;  // event not resolved (the call fails or retries)

// ---- one call's control block -------------------------------------------------------
// Words of a device buffer: the ingest's counters, stamps of the device's fixed-rate clock
// (one kernel at each phase's start writes its own: an event between kernels costs a small
// call 3 us), the emission's and the trie's control words, then the scan's block sums.
constexpr int kCtlCounters = 0, kCtlStamps = 8, kCtlCanon = 16, kCtlTrie = 24, kCtlSums = 32;
// call start, ingest, collection, ordering, node arrays; the end is stamped by launch_finish
enum Stamp { kStampCall = 0, kStampIngest = 1, kStampCollect = 2, kStampOrder = 3, kStampNodes = 4, kStampEnd = 5 };
__device__ inline void stamp(unsigned long long *at) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *at = (unsigned long long)wall_clock64();
}

// ---- path hashing ----------------------------------------------------------------
// Checkpoint hashes (prefixes at 16-frame boundaries, used to order paths) are a sum
// over the frames of a term of (frame, position), so partial sums over any split of
// the path combine by addition; a murmur3-style finalizer mixes in the length.  The
// term is one 32 x 32 -> 64-bit product of two position-dependent mixes of the frame;
// both factors move with the position, so paths over a few small frame ids still
// spread.  Correctness never depends on a hash: every match is verified frame by frame.
constexpr uint32_t kTermMulX = 0x9E3779B9u, kTermMulY = 0x85EBCA6Bu, kTermXorY = 0x5BD1E995u;
__host__ __device__ inline uint64_t frame_term(uint32_t f, uint32_t k) {
  const uint32_t x = f + k * kTermMulX;
  const uint32_t y = (f ^ kTermXorY) + k * kTermMulY;
  return (uint64_t)x * (uint64_t)(y | 1u);
}
// The unique-path table hashes pairs of frames instead.  A path of len frames is cut
// into ceil(len / 16) blocks of 16 frames: block m starts at frame 16 m, except that
// the last block of a path of 16 frames or more ends at the path's end (so it overlaps
// the block before it when len is not a multiple of 16; a path shorter than 16 frames
// is one block, zero-padded).  Pair i of block m, (F[s + 2i], F[s + 2i + 1]) with s the
// block's first frame, is pair p = 8 m + i and contributes
//   (F[s + 2i] + p*kPairMulX + kPairAddX) * (F[s + 2i + 1] + p*kPairMulY + kPairAddY)
// (factors wrap at 32 bits; the product and the sum at 64).  Unless its first factor
// is zero the term is injective in the second frame, both factors move with the
// position, and it costs one 32 x 32 -> 64-bit multiply-add per two frames; and every
// block but a short path's single one holds 16 frames of the path, so hashing it needs
// no mask.  (A collision costs only time: every table match is verified frame by
// frame.)
constexpr uint32_t kPairMulX = 0x9E3779B9u, kPairMulY = 0x85EBCA6Bu, kPairAddX = 0x27D4EB2Fu,
                   kPairAddY = 0x165667B1u;
__host__ __device__ inline uint64_t pair_term(uint32_t f0, uint32_t f1, uint32_t p) {
  const uint32_t x = f0 + p * kPairMulX + kPairAddX;
  const uint32_t y = f1 + p * kPairMulY + kPairAddY;
  return (uint64_t)x * (uint64_t)y;
}
// first frame of block m of a path of len frames (as above)
__host__ __device__ inline int64_t hash_block_start(int64_t m, int64_t len) {
  const int64_t s = 16 * m;
  return s + 16 > len && len >= 16 ? len - 16 : s;
}
__host__ __device__ inline uint64_t finish_hash(uint64_t s, uint64_t len) {
  uint64_t h = s + len * 0x9E3779B97F4A7C15ull;
  h ^= h >> 33;
  h *= 0xFF51AFD7ED558CCDull;
  h ^= h >> 33;
  h *= 0xC4CEB9FE1A85EC53ull;
  h ^= h >> 33;
  return h;
}

__device__ inline uint32_t hash32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7FEB352Du;
  x ^= x >> 15;
  x *= 0x846CA68Bu;
  x ^= x >> 16;
  return x;
}

// ---- arguments -----------------------------------------------------------------------
struct IngestArgs {
  // input batch
  const int64_t *off;
  const uint32_t *fr;
  int64_t n_events, n_frames;
  // unique-path table
  Slot *slot;
  uint64_t cap_mask;
  uint64_t hash_mask;   // all ones, except under a forced-collision test setting
  uint32_t *slot_of;    // [N] output: table slot of every event
  // the tree's path store (for paths seen in earlier calls)
  const uint32_t *pframes;
  const int64_t *pstart;
  const uint32_t *plen;
  // counters [kCtrCount]
  unsigned long long *ctr;
};

// What a call clears before its ingest, in one launch: the control block, the batch sums,
// the staging's counts (n_count may be 0), and a fresh table's slots (n_slots may be 0).
struct InitArgs {
  Slot *slot;
  uint64_t n_slots;
  uint64_t *delta;
  uint64_t n_delta;          // words
  uint32_t *count;
  uint64_t n_count;
  unsigned long long *ctl;
  uint64_t n_ctl;            // words
  int first;                 // the call's first attempt (stamps its start)
};
void launch_init(const InitArgs &a, hipStream_t s);
// n < 64 words from `from` into pinned host memory, and the clock after them
void launch_report(const unsigned long long *from, int n, unsigned long long *host, hipStream_t s);
void launch_finish(unsigned long long *ctl, unsigned long long *host, hipStream_t s);

// Host-side launch wrappers (one translation unit per kernel family).
void launch_ingest(const IngestArgs &a, int grid, hipStream_t s);
// Sum metrics [N][m] into delta[slot_of[e]][m] (delta starts zeroed).  Every workgroup
// sums its event range into an LDS map keyed by slot; the maps are flushed into
// staging buckets (bucket = slot >> bshift, plain stores, one counter atomic per
// bucket and workgroup), and one workgroup per bucket then adds the bucket's staged
// sums into delta.  Entries that find no room (LDS map full, bucket full) are added
// to delta with atomics.
struct AggStage {
  int32_t bshift;        // bucket of slot s: s >> bshift (agg_bucket_shift(m))
  int64_t nbuckets;      // 0: no staging (maps flushed with atomics)
  int64_t bucket_cap;    // staged entries per bucket
  uint32_t *count;       // [nbuckets], zeroed before the launch
  uint32_t *keys;        // [nbuckets][bucket_cap]
  uint64_t *sums;        // [nbuckets][bucket_cap][m]
};
int agg_bucket_shift(int32_t m);
int64_t agg_max_buckets();
int64_t agg_map_entries(int32_t m);
void launch_aggregate(const uint32_t *slot_of, const uint64_t *w, int64_t n, int32_t m, uint64_t *delta,
                      uint64_t cap, int grid, const AggStage &st, hipStream_t s);
// List the slots claimed in this call (word ref with kEventRef): new_slots, each new
// path's first frame in the batch and length (src_len, two words per path) and its place
// in the store relative to the frames already there (starts, 16-frame aligned, growing
// with the list position), and into ctr: kCtrNew (count << kNewShift | 16-frame blocks of
// store), kCtrNewLen (sum of lengths).  new_slots, src_len and starts hold room for list_cap
// paths, every possible new one: min(cap, events of the batch).  A batch of N <= CCT_MAX_EVENTS events
// has fewer than 2^31 new paths; the blocks of its new paths must fit kNewShift bits
// (2^37 frames and more than a GPU holds).
constexpr int kNewShift = 33;
constexpr unsigned long long kNewBlocksMask = (1ull << kNewShift) - 1;
void launch_collect_new(const Slot *slot, uint64_t cap, const int64_t *off, uint32_t *new_slots, int64_t *src_len,
                        uint64_t *starts, int64_t list_cap, unsigned long long *ctl, hipStream_t s);

// Path store: path d occupies frames [pstart[d], pstart[d] + round16(plen[d])) of
// pframes (pstart is a multiple of kStoreAlign, the tail is zero-filled), and its
// checkpoint hashes cp[pstart[d] / kStoreAlign + b] = hash of its prefix of length
// kStoreAlign * (b + 1), for every full block b.
constexpr int kStoreAlign = 16;
__host__ __device__ inline int64_t round_store(int64_t len) {
  return (len + kStoreAlign - 1) / kStoreAlign * kStoreAlign;
}

struct PublishArgs {
  const int64_t *off;        // batch offsets (frames of new paths come from the batch)
  const uint32_t *fr;
  int64_t n_frames;          // frames in the batch
  Slot *slot;
  const uint32_t *new_slots;
  int64_t n_new;
  int64_t d_old;
  uint32_t *pframes;
  uint64_t *pcp;             // checkpoint hashes
  int64_t *pstart;
  uint32_t *plen;
  uint32_t *pslot;
  int64_t store_used;        // frames already used in the store
  const uint64_t *starts;    // [n_new] place of each new path past store_used
  const int64_t *src_len;    // [n_new][2] first frame in the batch and length of each new path
  uint64_t *bpos;            // block positions for the trie (see TrieArgs), or null
  unsigned long long *empty; // set to 1 if the empty path is new (with bpos)
  uint64_t cp_mask;          // all ones, except under a test setting that forces collisions
};
void launch_publish(const PublishArgs &a, hipStream_t s);
// Exclusive prefix sums of `rows` rows of C uint64 columns (mod 2^64) into out[0..rows),
// totals into out row `rows`; blk holds (rows / 1024 + 1) * C scratch words.
void launch_scan(const uint64_t *in, int64_t rows, int C, uint64_t *blk, uint64_t *out, hipStream_t s);
// slot[list[i]] = empty for i < n (the slots published by a call that failed afterwards)
void launch_reset_slots(Slot *slot, const uint32_t *list, int64_t n, hipStream_t s);
void launch_unclaim(Slot *slot, uint64_t cap, hipStream_t s);
void launch_rehash(const uint32_t *pframes, const int64_t *pstart, const uint32_t *plen, int64_t d,
                   Slot *slot, uint64_t cap_mask, uint64_t hash_mask, uint32_t *pslot, hipStream_t s);

constexpr int kSortBlock = 1024;   // paths per block-local sort
struct alignas(16) CanonRec {  // the path at a canonical position
  int64_t start;         // first frame in the store
  uint32_t len, lcp;     // length, LCP with the path before it
};
struct CanonArgs {
  int64_t d;             // number of distinct full paths
  // the sort kernels order path ids id0 .. id0 + d - 1 by path (0 for a full sort), or a
  // merge's new ones by (gap[id - id0], path)
  int64_t id0;
  const uint32_t *gap;
  uint64_t few_gaps;     // a large merge: sampled neighbours in one gap (u_out[2]) from which on comparing pays
  int32_t lcp_known;     // launch_canon: lcp holds what launch_merge_order knows already, kInf elsewhere
  int32_t m;
  int32_t exact;         // 1: compare frames only (no checkpoint-hash shortcut)
  const uint32_t *pframes;
  const uint64_t *pcp;
  const int64_t *pstart;
  const uint32_t *plen;
  // sums after the batch, written by launch_canon (a fresh array): old paths (d < d_old)
  // add their slot's delta to old_sums, new ones take it
  int64_t d_old;
  const uint32_t *pslot;
  const uint64_t *delta;     // [slots][m]
  const uint64_t *old_sums;  // [d_old][m]
  uint64_t *psums;           // [D][m]
  // outputs / scratch
  uint32_t *order;       // [D] path ids in lexicographic order
  uint32_t *order_tmp;   // [D]
  uint32_t *lcp;         // [D+1] lcp with the previous path in order; lcp[D] = 0 (room for a multiple of 16)
  CanonRec *rec;         // [D]
  uint64_t *scan_in;     // [D][1+m] new-node counts and sums in order
  uint64_t *scan_out;    // [D+1][1+m] exclusive prefix sums (+ totals at row D)
  uint64_t *scan_blk;    // [ceil(D / 1024)][1+m] sums of 1024 rows, zeroed before launch_canon
  // minima of lcp: level 0 is lcp itself, an entry of level 1 covers 16 positions, an entry
  // of every further level 64 of the one below (min_levels of them, until one group is
  // left); every level padded to a multiple of 16 entries
  uint32_t *mins[6];
  int64_t min_n[6];
  int32_t min_levels;
  uint32_t *chain_parent; // [D]
  uint32_t *win_path;    // [U_max / 64 + 1] path index (in order) holding each 64-node window's first node
  int64_t u_max;
  // node arrays
  uint32_t *parent, *frame, *depth;
  uint32_t *subend;      // [U] end of each node's subtree: its descendants are the ids (u, subend[u])
  uint64_t *excl, *incl;
  unsigned long long *u_out;  // device: [0] node count, [1] order-violation flag, [2] neighbours in one gap
  unsigned long long *stamps;
  int grid_nodes;
};
void launch_sort(CanonArgs &a, hipStream_t s);        // leaves the result in a.order
// Order after a merge: every path new in this call (ids d_old .. a.d - 1) finds its
// gap in the previous order (d_old ids, sorted; the old paths keep their relative
// order) by binary search, the new paths are sorted by (gap, path), and both lists
// are placed by integer arithmetic; the LCPs of old neighbours that stay neighbours are
// taken from old_lcp.  scratch: 4 words for every new path,
// rounded up to a multiple of kSortBlock.  Leaves the result in a.order.
void launch_merge_order(CanonArgs &a, const uint32_t *old_order, const uint32_t *old_lcp, int64_t d_old,
                        uint32_t *scratch, hipStream_t s);

// Lexicographic order of the D distinct paths through a trie of 16-frame blocks (see
// trie.hip).  Scratch sizes: nblocks = store blocks in use (sum of ceil(len / 16)),
// cap = power of two >= 2 * nblocks.
struct TrieArgs {
  int64_t d;
  int64_t nblocks;
  uint64_t cap;                // node table capacity (power of two)
  const uint32_t *pframes;
  const uint64_t *pcp;
  const int64_t *pstart;
  const uint32_t *plen;
  uint64_t *tkey;              // [cap] node keys (0: empty)
  uint32_t *tval;              // [cap] node id of each key: the store block that claimed it
  uint32_t *count;             // [cap] distinct paths through each key's node
  uint32_t *hist;              // [cap + 1] its children (entry cap: the root's)
  uint64_t *bpos;              // [nblocks] (path length << 32) | index of the block in its path
  uint32_t *oslot, *occ;       // [nblocks] table slot and node of each store block
  // per node (its id is a store block, its representative; id nblocks is the root, where an
  // array has nblocks + 1 entries)
  uint32_t *nparent;           // [nblocks] parent node
  uint32_t *ncount;            // [nblocks] distinct paths through the node
  uint32_t *nend;              // [nblocks] a path ends at the node
  uint32_t *nchild;            // [nblocks + 1] children, where there are any
  uint32_t *gstart;            // [nblocks + 1] position of a node's first child
  uint32_t *cidx;              // [nblocks] index of each node among its siblings (root's children:
                               //           (link workgroup << 22) | index within the workgroup)
  uint32_t *weight;            // [nblocks] what the node adds to the ranks of the paths through it
  uint32_t *place;             // [nblocks] (bucket << 24) | index there, for members of large groups
  uint32_t *rootbase;          // [1024] first index of each link workgroup's root children
  int32_t large;               // groups of more siblings are split into buckets (set by launch_trie_sort)
  uint32_t *grouped;           // [nblocks] nodes grouped by parent
  uint32_t *grouped2;          // [nblocks] the same with the large groups' nodes in their buckets
  uint64_t *unit, *unit2;      // [nblocks] (start << 32 | size) of each position's group, or bucket
  uint32_t *base2;             // [nblocks] paths in the buckets before it
  uint64_t *lists;             // [large_cap] (start << 32 | size) of the large groups
  int64_t large_cap;           // large groups that can be listed
  uint32_t *lgroup;            // [nblocks + 1] list index of a large group, by parent node
  uint32_t *spl;               // [large_cap][256] splitters (node ids)
  uint32_t *bcnt, *bsum;       // [large_cap][256] bucket sizes, path counts
  unsigned long long *ctr;     // [8], zeroed before
  unsigned long long *stamps;
  uint32_t *order;             // [D] out: path ids in lexicographic order
};
// large groups listed, an empty path seen, nodes, failure
constexpr int kTrieCtrLarge = 0, kTrieCtrEmpty = 1, kTrieCtrNodes = 2, kTrieCtrFail = 4;
// bpos of block k of a path of len frames
__host__ __device__ inline uint64_t make_bpos(uint64_t len, uint64_t k) { return (len << 32) | k; }
// ctr[kTrieCtrFail] != 0 after the call: the trie could not be used (the caller sorts
// another way).  bpos holds the blocks of the paths from d_old on (launch_publish).
void launch_trie_sort(const TrieArgs &a, int64_t d_old, hipStream_t s);
// Levels of the minima of n = D + 1 positions: their entries in min_n, the words of levels
// 1 and up as the result, and set_min_levels points mins at them (level 0 at lcp).
int64_t min_level_words(int64_t n, CanonArgs &a);
void set_min_levels(CanonArgs &a, uint32_t *words);
// n arrays of 4-byte words copied in one launch
struct CopyArgs {
  int n;
  const uint32_t *src[5];
  uint32_t *dst[5];
  uint64_t words[5];
};
void launch_copy(const CopyArgs &a, hipStream_t s);
void launch_canon(const CanonArgs &a, hipStream_t s);  // lcp, sums, minima, emission

struct alignas(32) PathRec {  // the path at a canonical position
  int64_t start;             // first frame in the store
  uint32_t len, lcp;         // length, common prefix with the path before it
  int64_t base;              // id of its first node (of depth lcp + 1)
  int64_t pad;
};
struct QueryArgs {
  int64_t q;
  int64_t qn_frames;
  const int64_t *qoff;
  const uint32_t *qfr;
  int64_t d;
  int64_t u;                 // node count (ids are < u)
  int32_t m;
  const uint32_t *pframes;
  const int64_t *pstart;
  const uint32_t *plen;
  const uint32_t *order;
  const uint32_t *lcp;       // [D+1]
  const uint64_t *scan_out;  // column 0 holds the node-id bases
  const uint64_t *excl, *incl;
  int64_t *node_ids;
  uint64_t *qexcl, *qincl;
  unsigned long long *err;   // [2]: [0] malformed offsets (nothing is looked up), [1] inconsistent tree
  PathRec *sorted;           // [D]
  uint64_t *qtab;            // prefix index [qcap][2] {key, (length << 32) | position}, or null
  uint64_t qcap_mask;
  uint64_t qhash_mask;       // test setting: keys keep only these bits (forced collisions)
};
// the records of `sorted`
void launch_sorted_paths(const QueryArgs &a, hipStream_t s);
// the prefix index of every node (qtab cleared to zero first)
void launch_query_index(const QueryArgs &a, hipStream_t s);
// offsets check of the query batch (err bit 0), run before any output is written
void launch_query_check(const QueryArgs &a, hipStream_t s);
// lookups: through the index when a.qtab is set, else by binary search
void launch_query(const QueryArgs &a, hipStream_t s);

// Correlation-ID join of an activity flush with the registered call paths (activity.hip)
enum : int32_t { kActCtrError = 0, kActCtrUnmatched = 1, kActCtrMin = 2, kActCtrMax = 3, kActCtrUsed = 4,
                 kActCtrStart = 5, kActCtrCount = 6 };  // (kActCtrStart: the clock at the join's start)
enum : uint32_t { kActBadOffsets = 1, kActRepeatedId = 2, kActTableFull = 4 };
struct alignas(16) CorrSlot {
  uint64_t key;    // correlation ID (valid once claim != 0)
  uint32_t claim;  // registry index + 1; 0: empty
  uint32_t pad;
};
struct ActivityArgs {
  int64_t n_reg;             // registered paths
  int64_t reg_n_frames;
  const int64_t *reg_off;    // [n_reg + 1]
  const uint64_t *reg_corr;  // [n_reg] correlation IDs
  // dense IDs (max - min < 4 n_reg): a direct table dtab[id - id_min] (registry index + 1,
  // 0: not registered); otherwise the hash table
  bool dense;
  uint64_t id_min, id_span;  // registered IDs lie in [id_min, id_min + id_span]
  uint32_t *dtab;            // [id_span + 1]
  uint64_t cap_mask;         // hash table capacity - 1 (capacity a power of two >= 2 n_reg)
  CorrSlot *table;           // [cap]
  int64_t n_rec;             // activity records
  const uint64_t *rec_corr;  // [n_rec]
  uint32_t *ref;             // [n_reg] 0, or 1 + the index of a record naming the path (its owner)
  unsigned long long *ctr;   // [kActCtrCount]
};
void launch_corr_range(const ActivityArgs &a, hipStream_t s);  // counters; min and max registered ID
// clear the table (table_bytes, room for a multiple of 16) and ref (likewise), validate the
// offsets, insert, repeated IDs
void launch_corr_table(const ActivityArgs &a, uint64_t table_bytes, hipStream_t s);
// join and per-path sums of the matched records; list: scratch of corr_join_grid(n_rec)
// stripes (n_rec + corr_join_grid * 256 entries suffice), cnt: [corr_join_grid(n_rec)]
int64_t corr_join_grid(int64_t n_rec);
void launch_corr_join(const ActivityArgs &a, const uint64_t *metrics, int32_t m, uint64_t *sums, uint64_t *list,
                      uint32_t *cnt, hipStream_t s);
void launch_compact_lengths(const ActivityArgs &a, uint64_t *rows, hipStream_t s);
// the batch of referenced paths: offsets [n_paths + 1], frames and metrics; src_start is
// scratch [n_paths]
void launch_compact_gather(const ActivityArgs &a, const uint32_t *reg_frames, const uint64_t *scan,
                           const uint64_t *sums, int32_t m, int64_t n_paths, int64_t n_frames, int64_t *off_out,
                           int64_t *src_start, uint32_t *fr_out, uint64_t *met_out, hipStream_t s);

// Bottom-up view (bottomup.hip).  Stable radix sort of uint32 (key, value) pairs by 8 bits
// a pass: hist [256 * radix_blocks(n)], offs [256 * radix_blocks(n) + 1], scan_blk for
// launch_scan over as many rows.  launch_radix_bits prepares the first pass and writes the
// bits in which any keys differ and the time to host[0 .. 1] (bits [radix_blocks(n) + 1]);
// launch_radix_first completes it with the values 1 .. n.
int64_t radix_blocks(int64_t n);
void launch_radix_bits(const uint32_t *keys, int64_t n, uint64_t *hist, unsigned long long *bits,
                       unsigned long long *host, hipStream_t s);
void launch_radix_first(const uint32_t *keys, int64_t n, const uint64_t *hist, uint64_t *offs, uint64_t *scan_blk,
                        uint32_t *keys_out, uint32_t *vals_out, hipStream_t s);
void launch_radix_pass(const uint32_t *keys, const uint32_t *vals, int64_t n, int shift, uint64_t *hist, uint64_t *offs,
                       uint64_t *scan_blk, uint32_t *keys_out, uint32_t *vals_out, hipStream_t s);
// The view of n > 0 nodes sorted by frame (K, V): group heads per tile [bu_tiles(n)]; tags [n]
// and the exclusive max-scan of the tiles' largest, blk [bu_tiles(n)] (first: scan of heads);
// frames [G], ex and in [G][m].
int64_t bu_tiles(int64_t n);
void launch_bu_heads(const uint32_t *K, int64_t n, uint64_t *heads, hipStream_t s);
void launch_bu_tag(const uint32_t *K, const uint32_t *V, const uint64_t *first, const uint32_t *subend, int64_t n,
                   uint64_t *tag, uint64_t *blk, hipStream_t s);
void launch_bu_sums(const uint32_t *K, const uint32_t *V, const uint64_t *tag, const uint64_t *blk, const uint64_t *excl,
                    const uint64_t *incl, int64_t n, int64_t G, int32_t m, uint32_t *frames, uint64_t *ex, uint64_t *in,
                    hipStream_t s);

// Ratio filters over the tree's nodes (filter.hip)
enum : int32_t { kDenOne = 0, kDenMetric = 1, kDenRoot = 2 };
struct FilterArgs {
  int64_t u;
  int32_t m;
  const uint64_t *excl, *incl;  // [U][m]
  const uint32_t *subend;       // [U]
  int32_t num_metric, num_excl;
  int32_t den_kind, den_metric, den_excl;
  int32_t op;                   // +1: ratio above the threshold, -1: below
  uint64_t thr_num, thr_den;
  int32_t leaves_only;
};
constexpr int kFilterTile = 2048;  // nodes per tile of the two passes
int64_t filter_tiles(int64_t u);
// The filter that allocates nothing keeps its mask, counts and offsets in a static device
// array of kFilterStaticBytes per GPU, enough for kFilterStaticTiles tiles.
constexpr int64_t kFilterStaticTiles = 15360;  // trees of up to 31,457,280 nodes
constexpr size_t kFilterStaticBytes = 4u << 20;
struct FilterScratch {
  uint64_t *mask;   // [tiles * kFilterTile / 64], a bit per node
  uint32_t *count;  // [tiles] matches
  uint64_t *pos;    // [tiles + 1] their exclusive scan, where it is needed
};
// writes the first `capacity` matches to out, their number to *total (device or pinned host
// memory) and, if times is not null, the clock at the start and when the last tile's matches
// are written to times[0..2)
void launch_filter(const FilterArgs &a, const FilterScratch &f, int64_t capacity, int64_t *out,
                   unsigned long long *total, unsigned long long *times, hipStream_t s);
// Device address of the current device's static array (looked up once per device), or
// nullptr if the lookup failed; and the array's parts at that address.
void *filter_static_scratch();
FilterScratch filter_static_layout(void *base);

// Per-path and per-node statistics (stats.hip)
struct StatStage {  // staged per-path statistics of a batch (nbuckets = 0: device atomics instead)
  int32_t bshift;       // bucket of path i: i >> bshift
  int64_t nbuckets;
  int grid;             // workgroups of the per-slot kernel
  int64_t map_entries;  // LDS map entries per workgroup
  uint32_t *ev_path;    // [N] misses (path indices): workgroup g's from its first event index on
  uint64_t *ev_w;       // [N][m]
  uint32_t *map_key;    // [grid][map_entries]
  uint64_t *map_rec;    // [grid][map_entries][1 + 3m]: count, min[m], sq[m][2]
  uint64_t *hist_ev, *hist_map;  // [nbuckets][grid] entries per bucket and workgroup
  uint64_t *off_ev, *off_map;    // their exclusive scans, [nbuckets * grid + 1]
  uint32_t *wg_count;   // [grid][2]: misses, map entries
  uint32_t *st_ev_path;  // bucketed misses [N], values [N][m]
  uint64_t *st_ev_w;
  uint32_t *st_map_key;  // bucketed map entries [grid * map_entries], records
  uint64_t *st_map_rec;
};
struct PathStats {  // kept per path: cnt [D], min [D][m], sq [D][m][2]
  uint64_t *cnt, *min, *sq;
};
struct NodeStatOut {  // any pointer may be null
  uint64_t *count_excl, *count_incl;  // [U]
  uint64_t *min_excl, *min_incl;      // [U][m]
  uint64_t *sumsq_excl, *sumsq_incl;  // [U][m][2]
  double *mean_excl, *mean_incl;      // [U][m]
  double *std_excl, *std_incl;        // [U][m]
};
struct NodeStatArgs {
  int64_t u, d;
  int32_t m;
  const uint64_t *scan_out;  // [d + 1][1 + m] of the canonical emission
  const uint32_t *order;     // [d] canonical position -> path
  const uint64_t *pcnt, *pmin, *psq;
  const uint32_t *subend;         // [u]
  const uint64_t *excl, *incl;    // [u][m]
  uint64_t *rows, *prefix;        // [d][1 + 4m], [d + 1][1 + 4m], canonical path order
  uint32_t *node_path;            // [u]: canonical position of the path that created the node
  uint64_t *cmin, *pre, *suf;     // [d][m]
  uint64_t *tab;                  // [levels][nblk][m], nblk = rmq_blocks(d)
  int64_t nblk;
  int levels;
  NodeStatOut out;
};
int64_t stats_staged_entries(int32_t m);
int stats_bucket_shift(int32_t m);  // largest bucket: 2^shift paths
int64_t stats_max_buckets();
// slot -> path map for paths [0, D); paths [d_old, D) set to no sample
void launch_stats_prepare(int64_t D, int64_t d_old, int32_t m, const uint32_t *pslot, uint32_t *path_of_slot,
                          const PathStats &p, hipStream_t s);
void launch_stats_agg(const uint32_t *slot_of, const uint32_t *path_of_slot, const uint64_t *w, int64_t n, int32_t m,
                      int64_t D, int grid, const PathStats &p, const StatStage &st, uint64_t *scan_blk, hipStream_t s);
int64_t rmq_blocks(int64_t u);
void launch_node_stats(const NodeStatArgs &a, uint64_t *scan_blk, hipStream_t s);

}  // namespace cct
