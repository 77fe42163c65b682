// Embedding backward fused with the sparse SGD row update (transpose of Eq. (2);
// SGD of Sec. 5.1):  for every distinct row r looked up in table k,
//   g = sum_{p : idx_k[p] = r} dS[bag(p), k, :],   W_k[r,:] <- W_k[r,:] - lr * g.
//
// SORT path (deterministic, any table dtype) -- a most-significant-digit partition
// followed by a bucket-local sort, so that one workgroup owns all lookups of a row:
//   1. bucket_hist    : per 4096-position tile, histogram of the top digit of the row id
//                       (tiles never straddle two tables)
//   2. scan           : (digit, tile) counts -> destination offsets inside the table's slice
//                       (folded into step 3 when the batch has few tiles)
//   3. bucket_scatter : derives the bag of every position from the offsets, then moves the
//                       (row, bag) pairs to their bucket, stably, staged through LDS.
//                       Weighted batches (Eq. (2) with its weights) move (row, position) pairs
//                       instead and keep (bag, weight) records in a side array in the original
//                       order: nothing downstream looks inside the second member until a gradient
//                       row is fetched, where bag and weight are looked up by position.
//   4. bucket_reduce  : one workgroup per (table, top digit): stable LSD radix sort of the
//                       bucket on the remaining low bits (in LDS when it fits), run heads,
//                       then a lane group per run sums its dS rows in ascending position
//                       order (fp32) and read-modify-writes the table row once.  Runs longer
//                       than 32 are summed by the whole workgroup; runs longer than 2048 are
//                       queued per table as hot rows.  Buckets too large for LDS first split
//                       off their dominant rows unsorted (4a); what still does not fit goes to
//   4b. segment_sort / segment_reduce : a large list sorted by one workgroup per 2048 pairs
//                       with per-row counters in LDS, then reduced window by window.
//   5. hot_rows       : workgroup (bag group, table) sums the gradient rows of its bags for every hot
//                       row that names them: gathered (few hot rows), as a dense contraction on the
//                       matrix cores (multiplicity matrix [bag][hot row] times gradient tile), or,
//                       in weighted batches, from tiles staged in LDS.  The last workgroup of a table
//                       adds the partial sums in bag-group order and updates the rows.
// Steps 1-3 read indices and offsets only; dlrm_emb_bag_bwd_prepare enqueues just them.
// ATOMIC path (fp32 tables): a lane group per bag adds -lr*dS[b,k,:] to every row of the bag
// with hardware fp32 atomics; no workspace, one launch.  Measured 6x slower than SORT on the
// 8 x 1M x 64 multi-hot workload, so AUTO always takes SORT.
//
// Files: bwd_common.h (this: constants, workspace, arguments, shared device helpers),
// bwd_partition.hip (steps 1-3), bwd_sort.h (bucket and segment sorts), bwd_reduce.h (steps 4, 4a and
// the row updates; instantiated per optimizer in bwd_reduce_sgd.hip / bwd_reduce_adagrad.hip),
// bwd_tail.hip (segment sort, hot rows and their updates), bwd_export.hip (grouping exported for tests),
// emb_bwd.hip (entry points, ATOMIC path).
#pragma once
#include "common.h"

namespace dlrm {

constexpr int kThreads = 256;
constexpr int kNW = kThreads / DLRM_WAVE;       // wavefronts per workgroup
constexpr int kItems = 16;                      // positions per thread in a (large) partition tile
constexpr int kTile = kThreads * kItems;        // 4096 positions per tile; batches below kSmallTileNnz lookups
constexpr int kSmallItems = 4;                  // use tiles of 1024: four times the workgroups, a quarter of the
constexpr int64_t kSmallTileNnz = 1 << 20;      // dependent steps each (the partition of a small batch is a chain
                                                // of latencies on a mostly idle machine)
// log2 of the partition tile for a batch of nnz lookups (host and device agree through GroupArgs::tile_shift)
inline int tile_shift_for(int64_t nnz) { return nnz < kSmallTileNnz ? 10 : 12; }
constexpr int kMaxTopBits = 10;                 // partition digit: up to 1024 buckets per table
constexpr int kMaxBuckets = 1 << kMaxTopBits;
constexpr int kDPT = kMaxBuckets / kThreads;    // partition digits owned by one thread
constexpr int kSortBits = 8;                    // digit of the bucket-local LSD passes
constexpr int kSortBuckets = 1 << kSortBits;
constexpr int kBktItems = 8;                    // positions per thread in a bucket-sort tile
constexpr int kBktCap = kThreads * kBktItems;   // 2048: buckets up to this size are sorted in LDS
constexpr int kLongRun = 32;                    // longer runs are summed by the whole workgroup
constexpr int kBigMin = 256;                     // smallest bucket size that can count as heavy (see GroupArgs::big)
constexpr int kLongRunMin = 16;                 // ... 16 where a workgroup has >= 32 lane groups
constexpr int kHugeRun = 2048;                  // longer runs are split over workgroups
constexpr int kHotTileFloats = 16384;            // 64 KB of LDS: gradient rows of one bag tile
constexpr int kHotZeroRow = 256;                // floats of the widest gradient row
constexpr int kHotStagePasses = 16;             // float4 registers per thread holding the next tile
constexpr int kHotTilesPerGroup = 8;            // bag tiles streamed by one workgroup, at most
constexpr int kHotRunsPerWave = 8;              // hot runs a wavefront accumulates at once
constexpr int kFusedScanMaxTiles = 512;         // fold the scan into the scatter below this
constexpr int kSegMaxBits = 13;                 // oversized buckets with at most this many low bits are
                                                // sorted by many workgroups (per-row counters in LDS)
constexpr int kSegKeys = 1 << kSegMaxBits;
constexpr int kSmallBatch = 65536;              // up to this many lookups the three launches that only serve
                                                // oversized buckets and hot rows (4.5 us each with nothing to
                                                // do) are left out: a workgroup does that work in place
// Up to this many lookups per table on average a batch of at most kSmallBatch lookups is not partitioned at all: a
// bucket's workgroup picks its pairs out of the table's lookups (direct_reduce_kernel).  Update with / without a
// partition, one table of 1024, 4096 lookups (d = 64): 23.1 / 12.2, 23.0 / 14.1 us; 4 and 16 tables of 4096: 23.8 / 14.7,
// 28.4 / 20.3 us; 26 x 2048 one-hot (d = 16): 24.7 / 12.5 us.  The line was drawn where a single table's cost crossed
// (16384 lookups, row ids then passed 2048 at a time: 21.3 / 21.3 us), with room for tables above the mean.
// The rule sees the mean only (the host does not know the tables' counts), the cost is that of the longest table.  Batches
// with one long table among short ones, partitioned / not (d = 64): 26 x 2048 with 10240 in one 34 / 24 us, 8 x 512 with
// 28000 42 / 38 us, 16 x 1000 with 45000 57 / 57 us; where the long table's buckets outgrow the LDS sort as well the
// partition is ahead: 16 x 100 with 60000 128 / 153 us, 64 x 256 with 40000 325 / 415 us, 300 x 64 with 45000 1716 / 1897 us.
constexpr int kDirectPerTable = 4096;
constexpr int kRouteWords = 8;                  // words a workgroup keeps its route counters in (GroupArgs::direct)
constexpr int kCandMin = 128;                   // a row with this many of an oversized bucket's first
                                                // kBktCap pairs is split off before any sorting
constexpr int kCand = kBktCap / kCandMin;       // at most this many such rows
constexpr int kDenseFrom = 8;                   // tables with at least this many hot rows (unweighted batch)
                                                // have them summed as a dense contraction on the matrix cores
// Route counters of an update, kept behind the two segment counters in seg_meta (zeroed by the
// partition, read back by dlrm_emb_bag_bwd_route_counts): how often each rarely taken route ran.
constexpr int kRouteDirect = 2;                 // 1 after an update without a partition: the counters lie bucket by
                                                // bucket in hist, kRouteWords words each, laid out like seg_meta
                                                // (kRouteHeavy, kRouteOver: the bucket is heavy / oversized)
constexpr int kRouteHeavy = 2, kRouteOver = 3;
constexpr int kHotTables = 3;                   // with a partition: tables with hot rows
constexpr int kRouteSplit = 4;                  // oversized buckets that split off dominant rows
constexpr int kRouteGlobalSort = 5;             // lists sorted by one workgroup through global memory
constexpr int kRouteOneRow = 6;                 // oversized buckets holding a single row
constexpr int kRouteHugeInPlace = 7;            // runs above kHugeRun summed by one workgroup (no tail launches)

// ---------------------------------------------------------------------------
// Workspace layout (all offsets 256-byte aligned).  Arrays with several users hold, in the order of an update:
//   keys[0]            partition: digit_total from the column scan to the scatter; reduce: pair buffer 0
//   hist               partition: tile counts and, behind them, tile records (at 1024 digits: in vals[0]); update without a partition: route counters; weighted hot rows: partial sums
//   tile_heads         segment sort and hot rows: hot_done
//   seg_start, seg_tbl weighted: PosEntry records, all update long; unweighted hot rows: partial sums
// The exported grouping uses the last three as named, and runs no reduce.
struct WsLayout {
  size_t keys[2], vals[2];   // uint32[nnz] ping-pong: row ids / bag ids
  size_t hist;               // uint32[nt_max][1 << top_bits] (room for kMaxBuckets): per-tile digit counts / offsets
  size_t bucket_start;       // uint32[K * kMaxBuckets + 1]
  size_t tile_heads;         // uint32[nt_max + 1]
  size_t seg_start;          // uint32[nnz + 1]
  size_t seg_tbl;            // uint32[nnz], adjacent: seg_start and seg_tbl also serve as one array of nnz 8-byte entries
  size_t n_seg;              // uint32[4]            (export only)
  size_t huge_ctr;           // uint32[4]: [2] = listed (heavy) buckets, [3] = oversized buckets among them
  size_t hot_cnt;            // uint32[K]: queued hot runs per table
  size_t over_list;          // uint32[nnz / kBigMin + 1]: heavy buckets, handed to the first workgroups
  size_t segs;               // SegInfo[nnz / kBktCap + 2]: those of them sorted by many workgroups
  size_t seg_meta;           // uint32[8]: segment tiles, segments, kRouteDirect, kHotTables, route counters (kRoute*)
  size_t huge_runs;          // HugeRun[nnz / kHugeRun + K]: table k's list starts at sum_{j<k}(nnz_j/kHugeRun + 1)
  size_t huge_part;          // float[max_runs * bag groups * d], where more groups fit nowhere else (launch_hot)
  size_t total;
  int64_t nt_max;            // upper bound on the number of tiles
  int64_t max_huge;          // upper bound on the number of queued runs
};

// Weighted batches: what one lookup contributes besides its row, found by its position with one
// 8-byte load.
struct alignas(8) PosEntry {
  uint32_t bag;
  float w;  // the weight a of Eq. (2)
};

struct SegInfo {
  uint32_t start, n, k, low_bits;   // an oversized bucket: global position, pairs, table, unsorted bits
  uint32_t tile0, src, pad1, pad2;   // index of its first kBktCap-position tile among all segments;
                                     // pair buffer holding the unsorted pairs
};

struct HugeRun {
  uint32_t k, row, start, len;   // start: global position of the run's first sorted entry
  uint32_t pad0, src, pad1, pad2; // src: pair buffer holding the run
};

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// bags whose gradient rows one weighted hot-row workgroup streams at most: kHotTilesPerGroup tiles of
// kHotStagePasses passes of kThreads / G rows (G lanes per row)
inline int hot_group_bags(int d) { return kThreads / pow2_ceil(d / 4) * kHotStagePasses * kHotTilesPerGroup; }
inline int hot_groups(int B, int d) {
  const int gb = hot_group_bags(d);
  return (int)(((int64_t)B + gb - 1) / gb);
}

inline WsLayout ws_layout(int32_t K, int32_t B, int32_t d, int64_t nnz) {
  WsLayout L;
  size_t o = 0;
  const size_t n = (size_t)(nnz > 0 ? nnz : 1);
  L.nt_max = (nnz >> tile_shift_for(nnz)) + K;
  L.max_huge = nnz / kHugeRun + K;
  for (int i = 0; i < 2; ++i) { L.keys[i] = o; o = align256(o + n * 4); }
  for (int i = 0; i < 2; ++i) { L.vals[i] = o; o = align256(o + n * 4); }
  L.hist = o;         o = align256(o + (size_t)kMaxBuckets * (size_t)L.nt_max * 4);
  L.bucket_start = o; o = align256(o + ((size_t)K * kMaxBuckets + 1) * 4);
  L.tile_heads = o;   o = align256(o + (size_t)(L.nt_max + 1) * 4);
  L.seg_start = o;    o = align256(o + (n + 1) * 4);
  L.seg_tbl = o;      o = align256(o + n * 4);
  L.n_seg = o;        o = align256(o + 16);
  L.huge_ctr = o;     o = align256(o + 16);
  L.hot_cnt = o;      o = align256(o + (size_t)K * 4);
  L.over_list = o;    o = align256(o + ((size_t)(nnz / kBigMin) + 1) * 4);
  L.segs = o;         o = align256(o + ((size_t)(nnz / kBktCap) + 2) * sizeof(SegInfo));
  L.seg_meta = o;     o = align256(o + 32);
  L.huge_runs = o;    o = align256(o + (size_t)L.max_huge * sizeof(HugeRun));
  L.huge_part = o;    o = align256(o + (size_t)L.max_huge * (size_t)hot_groups(B, d) * (size_t)d * 4);
  L.total = o;
  return L;
}

// What the histogram kernel leaves for the scatter about a tile: one 32-byte load instead of the tile map and the
// search for the tile's first bag, which the histogram does while its row ids are on their way.
struct alignas(32) TileRec {
  uint32_t k, t, t0, nt;      // as in TileInfo
  uint32_t count;             // positions in the tile, 0: no tile
  uint32_t tbl_start;
  uint32_t shift;             // of the partition digit
  uint32_t bag;               // the bag that holds the tile's first position
};

// ---------------------------------------------------------------------------
struct GroupArgs {            // everything the grouping kernels need
  const void* indices;        // int64 or int32 (idx32)
  const int64_t* offsets;
  const int64_t* tbl_off;
  const int64_t* rows;
  int32_t idx32;
  const float* weights;       // NULL, or the weight of every lookup (parallel to indices)
  PosEntry* pos_entry;        // weighted batches: bag and weight of every position, in the original order
  int32_t K, B;
  int64_t nnz;                // lookups of all tables
  int64_t max_huge;           // upper bound on the queued hot runs of all tables
  int32_t nt_max;
  int32_t tile_shift;         // log2 of the positions per partition tile (10 or 12)
  int32_t top_bits;           // bits of the partition digit (0..kMaxTopBits)
  int32_t by_die;             // buckets dealt to the dies by table (bucket_id_of_block)
  int32_t fused_scan;         // 1: the scatter derives its offsets from the raw tile counts
  int32_t direct;             // 1: no partition, every bucket's workgroup picks its pairs out of the batch
  int32_t no_tail;            // 1: small batch, the segment and hot-row launches are left out and
                              //    bucket_reduce handles whatever they would have taken
  uint32_t* keys[2];
  uint32_t* vals[2];
  uint32_t* hist;
  TileRec* tile_rec;          // [nt_max], between the histogram and the scatter
  uint32_t* digit_total;      // [K << top_bits] pairs per bucket, between the column scan and the scatter
  uint32_t* bucket_start;
  uint32_t* tile_heads;
  uint32_t* seg_start;
  uint32_t* seg_tbl;
  uint32_t* n_seg;
  uint32_t* hot_cnt;
  uint32_t* hot_done;         // [K] workgroups that have left their partial sums of table k's hot rows
  uint32_t* list_cnt;         // heavy buckets listed by the partition (more than `big` pairs)
  uint32_t* over_cnt;         // those of them with more than kBktCap pairs (oversized)
  uint32_t* over_list;
  int32_t max_over;           // workgroups reserved at the front of the bucket grid for the listed buckets
  uint32_t big;               // a bucket with more pairs is heavy: 4 x the mean bucket, within [kBigMin, kBktCap]
  SegInfo* segs;
  int32_t seg_tiles_max;      // upper bound on the number of segment tiles
  uint32_t* seg_meta;         // [0] segment tiles, [1] segments (one 64-bit counter)
  HugeRun* huge_runs;
  float* huge_part;
};

// start of table k's hot-run list: every table may queue at most nnz_k / kHugeRun runs
__device__ inline uint32_t hot_list_base(const GroupArgs& a, int k) {
  uint32_t base = 0;
  for (int j = 0; j < k; ++j) base += (uint32_t)((a.tbl_off[j + 1] - a.tbl_off[j]) / kHugeRun) + 1u;
  return base;
}

// bits needed to index m rows; the partition digit of table k is row >> top_shift(k)
__device__ inline int key_bits(int64_t m) { return m <= 1 ? 0 : 64 - __clzll((unsigned long long)(m - 1)); }
__device__ inline int top_shift(const GroupArgs& a, int k) {
  const int s = key_bits(a.rows[k]) - a.top_bits;
  return s > 0 ? s : 0;
}

// Which table and which positions a tile covers.  Workgroup-uniform.
struct TileInfo {
  int k;
  int t;           // tile index inside the table
  int t0;          // global index of the table's first tile
  int nt;          // tiles of the table
  int64_t start;   // global position of the tile's first item
  int count;       // items in the tile (1 .. tile size)
  int64_t tbl_start;
  int total_tiles; // tiles of all tables
};

// Every workgroup rebuilds the tile map from tbl_off (K is small): tables own
// ceil(nnz_k / tile) consecutive tiles.  All threads must call this (it synchronises).
__device__ inline bool find_tile(const GroupArgs& a, int tile, TileInfo& ti, uint32_t* smem) {
  __shared__ int res[4];
  const int64_t tsize = (int64_t)1 << a.tile_shift;
  if (threadIdx.x == 0) res[0] = -1;
  uint32_t carry = 0;
  for (int k0 = 0; k0 < a.K; k0 += kThreads) {
    const int k = k0 + threadIdx.x;
    uint32_t nt = 0;
    if (k < a.K) nt = (uint32_t)((a.tbl_off[k + 1] - a.tbl_off[k] + tsize - 1) >> a.tile_shift);
    uint32_t total;
    const uint32_t first = carry + block_exclusive_scan<kThreads>(nt, smem, &total);
    if (k < a.K && (uint32_t)tile >= first && (uint32_t)tile < first + nt) {
      res[0] = k;
      res[1] = (int)first;
      res[2] = (int)nt;
    }
    carry += total;
  }
  __syncthreads();
  ti.total_tiles = (int)carry;
  if (res[0] < 0) return false;
  ti.k = res[0];
  ti.t0 = res[1];
  ti.nt = res[2];
  ti.t = tile - ti.t0;
  ti.tbl_start = a.tbl_off[ti.k];
  ti.start = ti.tbl_start + ((int64_t)ti.t << a.tile_shift);
  const int64_t rem = a.tbl_off[ti.k + 1] - ti.start;
  ti.count = (int)(rem < tsize ? rem : tsize);
  return true;
}

// --- shared by steps 3 and 4: stable ranking of a tile by a digit ---------------------
// Wave w of the workgroup owns the contiguous positions [w*64*items, (w+1)*64*items) of
// the tile, item j < items of lane l being position w*64*items + j*64 + l (items <= ITEMS is
// workgroup-uniform: a tile that is not full is dealt evenly to the wavefronts, and nobody ranks
// items that do not exist).  Ranks inside a wave come from ballot matching; per-wave digit counters
// in LDS give the order across waves.
// On return rnk[j] is the item's rank among the items of its wave with the same digit that
// precede it, and wcnt[w][digit] the wave's count.  wcnt must be zero on entry.
// Bound by latency (a wavefront or three per SIMD): CH items are matched side by side, bit by bit, and no
// step of an item waits for an answer that the next item's needs: all lanes read the count of their digit
// before the first lane of each digit adds to it (LDS operations of a wavefront run in order), instead of one
// lane adding, waiting and passing the old count on (7.7 us of a 4096-position tile's 21).  Step before / after: 8 tables of
// 205 K lookups, pooling + update 276 / 270 us; 64 fp16 tables of 524 K lookups 2979 / 2901 us.
template <int ITEMS, int NBK, int CH = 4>
__device__ inline void rank_items(const uint32_t* dg, const bool* ok, int bits,
                                  uint32_t (*wcnt)[NBK], uint32_t* rnk, int items = ITEMS) {
  static_assert(ITEMS % CH == 0, "whole chunks");
  uint32_t* cnt = wcnt[wave_id()];
#pragma unroll
  for (int j0 = 0; j0 < ITEMS; j0 += CH) {
    if (j0 >= items) break;  // uniform
    // lo, hi: lanes of this wave holding the same digit in the item (meaningful where ok)
    uint32_t lo[CH], hi[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const unsigned long long v = __ballot(ok[j0 + c]);
      lo[c] = (uint32_t)v;
      hi[c] = (uint32_t)(v >> 32);
    }
    for (int bit = 0; bit < bits; ++bit) {
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const uint32_t one = (uint32_t)__builtin_amdgcn_sbfe((int)dg[j0 + c], (unsigned)bit, 1u);   // all bits set if it is
        const unsigned long long bal = __ballot(one != 0u);
        lo[c] &= ~((uint32_t)bal ^ one);
        hi[c] &= ~((uint32_t)(bal >> 32) ^ one);
      }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const uint32_t before = __builtin_amdgcn_mbcnt_hi(hi[c], __builtin_amdgcn_mbcnt_lo(lo[c], 0u));
      uint32_t* slot = cnt + dg[j0 + c];
      rnk[j0 + c] = before + __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __builtin_amdgcn_wave_barrier();   // every lane has read before the first of each digit adds
      if (ok[j0 + c] && before == 0u)
        __hip_atomic_fetch_add(slot, (uint32_t)(__popc(lo[c]) + __popc(hi[c])), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// After rank_items + a barrier: turns wcnt[w][digit] into the tile-local sorted position of
// wave w's first item with that digit.  Thread t owns the DPT = NBK/256 consecutive digits
// t*DPT .. t*DPT+DPT-1 and gets their tile-local offsets and counts.  All threads must call it.
template <int NBK>
__device__ inline void digit_offsets(int nb, uint32_t (*wcnt)[NBK], uint32_t* scan_smem,
                                     uint32_t* lofs_out, uint32_t* tot_out) {
  constexpr int DPT = NBK / kThreads;
  uint32_t c[DPT][kNW], tot[DPT], sum = 0;
#pragma unroll
  for (int q = 0; q < DPT; ++q) {
    const int dg = threadIdx.x * DPT + q;
    tot[q] = 0;
#pragma unroll
    for (int i = 0; i < kNW; ++i) {
      c[q][i] = dg < nb ? wcnt[i][dg] : 0u;
      tot[q] += c[q][i];
    }
    sum += tot[q];
  }
  uint32_t total_all;
  uint32_t run = block_exclusive_scan<kThreads>(sum, scan_smem, &total_all);
#pragma unroll
  for (int q = 0; q < DPT; ++q) {
    const int dg = threadIdx.x * DPT + q;
    lofs_out[q] = run;
    tot_out[q] = tot[q];
    if (dg < nb) {
#pragma unroll
      for (int i = 0; i < kNW; ++i) {
        wcnt[i][dg] = run;
        run += c[q][i];
      }
    }
  }
}

// Oversized buckets whose unsorted low bits fit per-row counters in LDS become "segments",
// sorted by one workgroup per kBktCap-position tile (segment_sort_kernel).  One workgroup builds
// the segment list and its tile map.  All threads call it.

struct Bucket {
  int k;
  uint32_t start, n;   // global position of the bucket's first pair, pairs in the bucket
  int low_bits;        // row-id bits below the partition digit
  uint32_t* route;     // route counters of its workgroup (kRoute*)
  float* H;            // the table's optimizer state (state_base)
};

// Heavy buckets (hot rows: long runs, or more pairs than the LDS sort holds) take much longer than
// the rest: they are listed during the partition and handed to the FIRST workgroups of the grid, so
// that they start at once and run beside everything else; the workgroup a heavy bucket would get by
// its index leaves it alone.  Returns false if this workgroup has nothing to do.
__device__ inline bool bucket_id_of_block(const GroupArgs& a, uint32_t* id, bool* listed) {
  if (blockIdx.x < (uint32_t)a.max_over) {
    if (blockIdx.x >= *a.list_cnt) return false;
    *id = a.over_list[blockIdx.x];
    *listed = true;
    return true;
  }
  // Workgroups go to the eight accelerator dies round-robin by their index, and every die has an L2 of
  // its own.  The gradient rows a bucket gathers belong to its table alone, so with large gradient
  // slices (by_die) a die works through whole tables (die x: tables x, x + 8, ...) and its L2 holds one
  // table's slice at a time, not an eighth of the buckets of every table.  Tables past the last
  // multiple of 8 keep the plain order.
  const uint32_t j = blockIdx.x - (uint32_t)a.max_over;
  const uint32_t k8 = (uint32_t)a.K & ~7u;
  if (a.by_die && j < (k8 << a.top_bits)) {
    const uint32_t die = blockIdx.x & 7u, q = j >> 3;
    *id = ((((q >> a.top_bits) << 3) + die) << a.top_bits) | (q & ((1u << a.top_bits) - 1u));
  } else {
    *id = j;
  }
  *listed = false;
  return true;
}

__device__ inline Bucket bucket_of_block(const GroupArgs& a, uint32_t id) {
  const int nb = 1 << a.top_bits;
  Bucket b;
  b.k = (int)(id >> a.top_bits);
  const int dg = (int)(id & (uint32_t)(nb - 1));
  b.start = 0;
  b.n = 0;
  b.low_bits = 0;
  b.route = a.seg_meta;
  b.H = nullptr;
  if (a.tbl_off[b.k + 1] == a.tbl_off[b.k]) return b;  // no lookups: its bucket_start is never written
  b.start = a.bucket_start[(size_t)b.k * nb + dg];
  const uint32_t end = dg + 1 < nb ? a.bucket_start[(size_t)b.k * nb + dg + 1] : (uint32_t)a.tbl_off[b.k + 1];
  b.n = end - b.start;
  b.low_bits = top_shift(a, b.k);
  return b;
}

struct UpdArgs {
  void* const* tables;
  void* const* state;   // Adagrad: K fp32 accumulators shaped like the tables; else unused
  const float* dS;
  int64_t stride_b, stride_k;
  float lr, eps;
  int32_t d;
};

// What is done to a row once its gradient g is summed (Sec. 5.1 names both optimizers):
//   kSgd     : W <- W - lr * g
//   kAdagrad : h <- h + g*g (fp32 state), W <- W - lr * g / (sqrt(h) + eps), element-wise
constexpr int kSgd = 0, kAdagrad = 1;

// Narrow rows that are not whole 64-byte sectors: a sector holds parts of two or more rows and a bucket's rows are
// neighbours, so plain loads find in the L2 what streaming ones fetch once per row.  Lookup + update, 8 tables of 1M rows,
// 1.6M lookups, three sets of tables in turn, streaming / plain loads, us: fp32 SGD, d = 12 180 / 177, 28 264 / 244,
// 36 294 / 290; Adagrad, d = 4 293 / 225, 36 524 / 468, 60 662 / 626; fp16 SGD, d = 24 182 / 183, 56 274 / 266 (0.2M
// lookups of 16 bytes: 72 / 62).  With plain stores as well: d = 28 250, 36 293, Adagrad 36 474, 60 657; whole sectors
// (d = 48 fp32, stores too): 259 / 303.  The limits leave out what was slower (plain stores too): fp32 SGD d = 52
// 341 / 356, 16-bit d = 72 306 / 313, 16-bit Adagrad d = 56 475 / 488.
// The rule sees the width alone; where few neighbours are looked up plain loads are no slower either.  Lookup + update, two sets in
// turn, lookups per row 0.2 / 0.02 / 0.002 / 2 (8 x 1M, 4 x 10M twice, 8 x 0.1M rows): fp32 SGD d = 12 170 / 163, 115 / 105,
// 37.1 / 35.9, 105 / 98; Adagrad d = 36 515 / 442, 302 / 268, 55.8 / 50.1, 268 / 253; fp16 SGD d = 24 172 / 169, 116 / 109,
// 36.2 / 34.9, 115 / 102.  Of 90 such pairs four are slower: fp16 SGD d = 40 213 / 222 and 136 / 139 (38.0 / 36.6 and 149 / 134
// the others), d = 56 161 / 163, fp32 SGD d = 36 173 / 177.  Small batches without a partition, 26 tables of 2000 lookups:
// fp32 SGD d = 36 25.1 / 22.3, Adagrad d = 4 22.0 / 18.5, fp16 SGD d = 40 22.9 / 21.3.
constexpr int keep_below(int dtype, int opt) {   // bytes of a row
  return dtype == DLRM_F32 ? (opt == kAdagrad ? 256 : 160) : (opt == kAdagrad ? 96 : 128);
}
inline bool rows_share_sectors(int d, int dtype, int opt) {
  const int bytes = d * elem_bytes(dtype);
  return bytes % 64 != 0 && bytes < keep_below(dtype, opt);
}

// The 4 columns [chunk*4, chunk*4+4) of a table row: raw load, and update + store
// (fp32: W - lr*g; fp16/bf16: widen, update in fp32, one round-to-nearest-even).
// W: base of the table, read from the pointer array ONCE per workgroup -- the row stores below
// may alias anything as far as the compiler knows, so a per-row read of tables[k] would be
// re-issued (and waited for) before every row.
template <int DT>
__device__ inline char* row_chunk_ptr(char* W, int d, uint32_t row, int chunk) {
  return W + ((int64_t)row * d + chunk * 4) * Tab<DT>::EB;
}
// KEEP: plain loads that stay in the caches, for narrow rows that share 64-byte sectors (rows_share_sectors); else streaming.
template <int DT, bool KEEP = false>
__device__ inline u32x4 row_chunk_load(const char* p) {
  if constexpr (DT == DLRM_F32) {
    return KEEP ? load16(p) : load16_stream(p);
  } else {
    const u32x2 b = KEEP ? *reinterpret_cast<const u32x2*>(p) : load8_stream(p);
    return u32x4{b.x, b.y, 0u, 0u};
  }
}
template <int DT>
__device__ inline void row_chunk_update_store(char* p, u32x4 raw, f32x4 g, float lr) {
  if constexpr (DT == DLRM_F32) {
    f32x4 x;
    x.x = fmaf(-lr, g.x, u2f(raw.x));
    x.y = fmaf(-lr, g.y, u2f(raw.y));
    x.z = fmaf(-lr, g.z, u2f(raw.z));
    x.w = fmaf(-lr, g.w, u2f(raw.w));
    store16_stream(p, u32x4{f2u(x.x), f2u(x.y), f2u(x.z), f2u(x.w)});
  } else {
    float x0, x1, x2, x3;
    if constexpr (DT == DLRM_F16) {
      half2_to_float2(raw.x, x0, x1);
      half2_to_float2(raw.y, x2, x3);
    } else {
      bf162_to_float2(raw.x, x0, x1);
      bf162_to_float2(raw.y, x2, x3);
    }
    x0 = fmaf(-lr, g.x, x0);
    x1 = fmaf(-lr, g.y, x1);
    x2 = fmaf(-lr, g.z, x2);
    x3 = fmaf(-lr, g.w, x3);
    u32x2 b;
    if constexpr (DT == DLRM_F16) {
      b.x = float2_to_half2(x0, x1);
      b.y = float2_to_half2(x2, x3);
    } else {
      b.x = float2_to_bf162(x0, x1);
      b.y = float2_to_bf162(x2, x3);
    }
    store8_stream(p, b);
  }
}
// The same 4 columns of a row together with their optimizer state (none for SGD).
struct RowRef {
  char* w;
  float* h;
};
struct RowVal {
  u32x4 w;
  f32x4 h;
};
template <int DT, int OPT>
__device__ inline RowRef row_ref(char* W, float* H, int d, uint32_t row, int chunk) {
  const int64_t e = (int64_t)row * d + chunk * 4;
  RowRef r;
  r.w = W + e * Tab<DT>::EB;
  r.h = OPT == kAdagrad ? H + e : nullptr;
  return r;
}
template <int DT, int OPT, bool KEEP = false>
__device__ inline RowVal row_load(const RowRef& r) {
  RowVal v;
  v.w = row_chunk_load<DT, KEEP>(r.w);
  v.h = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (OPT == kAdagrad) {
    const u32x4 hb = KEEP ? load16(r.h) : load16_stream(r.h);
    v.h = f32x4{u2f(hb.x), u2f(hb.y), u2f(hb.z), u2f(hb.w)};
  }
  return v;
}
template <int DT, int OPT>
__device__ inline void row_update_store(const RowRef& r, const RowVal& v, f32x4 g, const UpdArgs& u) {
  if constexpr (OPT == kAdagrad) {
    f32x4 h, step;
    h.x = fmaf(g.x, g.x, v.h.x);
    h.y = fmaf(g.y, g.y, v.h.y);
    h.z = fmaf(g.z, g.z, v.h.z);
    h.w = fmaf(g.w, g.w, v.h.w);
    store16_stream(r.h, u32x4{f2u(h.x), f2u(h.y), f2u(h.z), f2u(h.w)});
    step.x = u.lr * g.x / (sqrtf(h.x) + u.eps);
    step.y = u.lr * g.y / (sqrtf(h.y) + u.eps);
    step.z = u.lr * g.z / (sqrtf(h.z) + u.eps);
    step.w = u.lr * g.w / (sqrtf(h.w) + u.eps);
    row_chunk_update_store<DT>(r.w, v.w, step, 1.0f);  // W - 1 * step, one rounding
  } else {
    row_chunk_update_store<DT>(r.w, v.w, g, u.lr);
  }
}
// A pointer that is the same in all lanes, as a scalar.
template <typename P>
__device__ inline P* uniform_ptr(P* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return reinterpret_cast<P*>(((uint64_t)hi << 32) | lo);
}
// Base of table k's optimizer state, read once per workgroup, like the table base, and held as a scalar.  As a vector
// load still on its way when the rows are requested, every request of a row waited for all requests before it:
// 13 fp32 tables of 36 columns, 0.5M lookups 155 / 135 us a step; 8 weighted ones of 64 columns, 0.8M lookups 259 / 244 us.
template <int OPT>
__device__ inline float* state_base(const UpdArgs& u, int k) {
  if constexpr (OPT == kAdagrad) return uniform_ptr(static_cast<float*>(u.state[k]));
  return nullptr;
}


// ---------------------------------------------------------------------------
int check_batch(const dlrm_sparse_batch* s);  // util.hip

// Bits of the partition digit, 1 << bits buckets a table, one workgroup to each: the fewest bits that leave a bucket no more pairs on
// average than a `buckets`-th of the batch, `most` where that is fewer, or 1024 where that is more.  (Bits halve a bucket: where
// `most` decides, a bucket has between half of it and all of it.)
inline int bits_for(int64_t nnz, int32_t K, double buckets, double most) {
  double target = (double)nnz / buckets;
  if (target < most) target = most;
  if (target > 1024.0) target = 1024.0;
  const double per_table = (double)nnz / (double)K;
  int tb = 0;
  while (tb < kMaxTopBits && per_table / (double)(1 << tb) > target) ++tb;
  return tb;
}
// 1536 buckets of 128 pairs for every width are the rule of small batches, whose split a batch without a partition shares
// (direct_reduce_kernel: every bucket reads all row ids of its table, 26 x 2048 one-hot 30 / 35 us with twice the buckets).
// Otherwise:
// Narrow rows.  A bucket is mostly its sort, so fewer and larger ones take less, 70 skewed tables of 2864 lookups, d = 4 51.9 / 44.6
// us an update, 50 uniform ones of 3526 37.7 / 32.7; but a hot row's bucket outgrows the LDS sort sooner, 13 skewed tables of
// 10540, d = 16 36.3 / 49.7.  They are taken where neither uniform nor skewed lookups lose on average over tables of one size and of
// sizes over three decades (6700 batches; mean of the update uniform / skewed of one size, of many, by the bits of 128 pairs): up to 4
// lanes 6 bits -12 / -9 %, -11 / +4, 10 -17 / -1, -16 / +1.  Not 7 -9 / -1, -8 / +13, 8 -11 / +4, -9 / +8, 9 -13 / +4, -11 / +5; 8 lanes
// 6 -9 / -5, -9 / +8, 7 -7 / +5, -9 / +8; 10 -13 / -2, -16 / -3.
// Wide rows.  A workgroup has few lane groups (four at 64 lanes), so a bucket of a given size takes it longer; one bit more, two at 64
// lanes, lets the buckets end together and leaves a hot row less company: 36 skewed tables of 20708, d = 96 186 / 149; 12
// uniform ones of 98814, d = 128 409 / 399; 36 skewed ones of 56105, d = 132 584 / 486.  The line is the mean bucket before the
// bit from which uniform lookups do not lose (13800 batches of 2^16 to 4 M lookups; of those with the bit uniform ones are 2 to 5 %
// ahead by width, skewed ones 8 to 13), beside a power of two rather than on it: 2^n samples with bags of 1..7 are 2^(n+2) lookups
// of a table but for a few, which would give the same program one digit and the other by turns.  It is higher
// - for 64 digits and fewer of 32 lanes, 79 uniform tables of 3785, d = 116 124.6 / 134.0;
// - where tables have fewer rows than lookups, which a bucket adds up in LDS, 8 uniform ones of 43048 and 1975 rows, d = 96 46.9 / 53.3;
// - for 512 digits (1024 at 64 lanes), every tile's counts growing with them, 8 uniform ones of 53677, d = 20 43.3 / 53.6; with more
//   rows than lookups 32 and 64 lanes do not lose by them (64 lanes, 310 batches 1024 digits / 512, uniform -1 %, skewed -4).
inline int digit_bits(int64_t nnz, int32_t K, int lanes, int64_t max_rows) {
  const int tb = bits_for(nnz, K, 1536.0, 128.0);
  if (nnz <= kSmallBatch) return tb;
  if (lanes <= 8 && (tb <= (lanes < 8 ? 6 : 5) || tb == kMaxTopBits)) {
    const int fewer = bits_for(nnz, K, 1536.0, lanes < 8 ? 224.0 : 192.0);
    if (fewer < tb) return fewer;
  }
  if (lanes < 8) return tb;
  const double per_table = (double)nnz / (double)K, full = (double)nnz / (lanes == 64 ? 4096.0 : 2560.0);
  const bool few_rows = per_table > (double)max_rows;
  int bits = tb;
  for (; bits < (lanes == 64 ? kMaxTopBits : kMaxTopBits - 1); ++bits) {
    const double mean = per_table / (double)(1 << bits);
    double least = lanes == 64 ? 112.0 : lanes == 32 ? (bits < 6 ? 160.0 : 112.0) : lanes == 16 ? 200.0 : (bits < 6 ? 240.0 : 400.0);
    if (few_rows && lanes < 64) least *= 1.5;
    if (bits + 1 > (lanes == 64 ? 9 : 8) && (few_rows || lanes < 32)) least *= 2.0;
    if (mean < least || mean <= full) break;
  }
  return bits;
}
// ... of a batch: never more than its row ids have
inline int partition_bits(int64_t nnz, int32_t K, int32_t d, int64_t max_rows) {
  const int tb = digit_bits(nnz, K, pow2_ceil(d / 4), max_rows), kb = ilog2_ceil(max_rows);
  return tb < kb ? tb : kb;
}

inline void fill_group_args(GroupArgs& g, const dlrm_sparse_batch* s, const WsLayout& L, void* ws) {
  char* base = static_cast<char*>(ws);
  g.indices = s->indices;
  g.idx32 = s->index_dtype == DLRM_I32;
  g.offsets = s->offsets;
  g.tbl_off = s->tbl_off;
  g.rows = s->rows;
  g.weights = s->weights;
  g.K = s->K;
  g.B = s->B;
  g.nnz = s->nnz_total;
  g.max_huge = L.max_huge;
  g.nt_max = (int32_t)L.nt_max;
  g.tile_shift = tile_shift_for(s->nnz_total);
  const int tb = partition_bits(s->nnz_total, s->K, s->d, s->max_rows);
  g.top_bits = tb;
  // Only for slices well above a die's 4 MB of L2 (measured: the hot-row workload's 8.4 MB slices -3.5 %
  // time and -21 % fetched bytes; 0.5 MB slices +8 % time), because a die then has whole tables and tables
  // differ in work: with 4 MB slices and tables of 100 to 10 M rows the kernel lost 15 %.
  g.by_die = (int64_t)s->B * s->d * 4 >= (6 << 20) ? 1 : 0;
  // the totals of the column scan lie in pair buffer 0, idle until the reduce; the batch has more lookups than
  // buckets unless it has more tables than lookups, whose few tiles each the scatter may as well add up itself
  g.fused_scan = L.nt_max <= kFusedScanMaxTiles || ((int64_t)s->K << tb) > s->nnz_total ? 1 : 0;
  g.no_tail = s->nnz_total <= kSmallBatch ? 1 : 0;
  g.direct = g.no_tail && s->nnz_total <= (int64_t)kDirectPerTable * s->K ? 1 : 0;
  for (int i = 0; i < 2; ++i) {
    g.keys[i] = reinterpret_cast<uint32_t*>(base + L.keys[i]);
    g.vals[i] = reinterpret_cast<uint32_t*>(base + L.vals[i]);
  }
  g.hist = reinterpret_cast<uint32_t*>(base + L.hist);
  g.digit_total = reinterpret_cast<uint32_t*>(base + L.keys[0]);
  // behind the tile counts, or, with the most digits, in pair buffer 0: 57344 lookups a table on average or more, 4 bytes each, and at
  // most a record of 32 bytes for 1024 of them and one a table
  const size_t counts = (((size_t)L.nt_max << tb) + 7) & ~(size_t)7;
  g.tile_rec = reinterpret_cast<TileRec*>(tb < kMaxTopBits ? base + L.hist + counts * 4 : base + L.vals[0]);
  g.bucket_start = reinterpret_cast<uint32_t*>(base + L.bucket_start);
  g.tile_heads = reinterpret_cast<uint32_t*>(base + L.tile_heads);
  g.seg_start = reinterpret_cast<uint32_t*>(base + L.seg_start);
  // the two export arrays, idle during an update and adjacent in the layout, hold the nnz records
  g.pos_entry = reinterpret_cast<PosEntry*>(base + L.seg_start);
  g.seg_tbl = reinterpret_cast<uint32_t*>(base + L.seg_tbl);
  g.n_seg = reinterpret_cast<uint32_t*>(base + L.n_seg);
  g.hot_cnt = reinterpret_cast<uint32_t*>(base + L.hot_cnt);
  g.hot_done = g.tile_heads;   // idle during an update, and holds more than K words
  g.list_cnt = reinterpret_cast<uint32_t*>(base + L.huge_ctr + 8);
  g.over_cnt = reinterpret_cast<uint32_t*>(base + L.huge_ctr + 12);
  g.over_list = reinterpret_cast<uint32_t*>(base + L.over_list);
  g.segs = reinterpret_cast<SegInfo*>(base + L.segs);
  g.seg_meta = reinterpret_cast<uint32_t*>(base + L.seg_meta);
  {
    const int64_t nbk = (int64_t)s->K << tb;
    int64_t big = 4 * (s->nnz_total / nbk);
    if (big < kBigMin) big = kBigMin;
    if (big > kBktCap) big = kBktCap;
    g.big = (uint32_t)big;
    const int64_t cap = s->nnz_total / big + 1, cap_over = s->nnz_total / kBktCap + 1;
    g.max_over = (int32_t)(nbk < cap ? nbk : cap);
    g.seg_tiles_max = (int32_t)(s->nnz_total / kBktCap + (nbk < cap_over ? nbk : cap_over));
  }
  g.huge_runs = reinterpret_cast<HugeRun*>(base + L.huge_runs);
  g.huge_part = reinterpret_cast<float*>(base + L.huge_part);
}

inline int check_ws(const dlrm_sparse_batch* s, void* ws, size_t bytes, WsLayout* L) {
  *L = ws_layout(s->K, s->B, s->d, s->nnz_total);
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255) || bytes < L->total) return DLRM_ERR_WORKSPACE;
  if (L->nt_max > 0x7FFFFFFF || ((int64_t)s->K << kMaxTopBits) > 0x7FFFFFFF) return DLRM_ERR_BAD_SHAPE;
  if (s->K > DLRM_MAX_BWD_TABLES) return DLRM_ERR_BAD_SHAPE;  // the hot-row launches put the table in grid.y
  return DLRM_OK;
}

// steps 1-3 (bwd_partition.hip): afterwards keys[1]/vals[1] hold the pairs partitioned into buckets
// and bucket_start the bucket boundaries
int enqueue_partition(const dlrm_sparse_batch* s, const GroupArgs& g, hipStream_t st);
// step 4 onwards with the SGD / Adagrad row update (bwd_reduce_sgd.hip, bwd_reduce_adagrad.hip)
// (one translation unit per optimizer and per weighted / unweighted pooling)
// tm: NULL, or the caller's event pair recorded around the bucket_reduce launch of this call
int run_reduce_sgd(const GroupArgs& g, const UpdArgs& u, int dtype, int G, int K, const dlrm_bwd_timing* tm,
                   hipStream_t st);
int run_reduce_adagrad(const GroupArgs& g, const UpdArgs& u, int dtype, int G, int K, const dlrm_bwd_timing* tm,
                       hipStream_t st);
int run_reduce_sgd_weighted(const GroupArgs& g, const UpdArgs& u, int dtype, int G, int K, const dlrm_bwd_timing* tm,
                            hipStream_t st);
int run_reduce_adagrad_weighted(const GroupArgs& g, const UpdArgs& u, int dtype, int G, int K,
                                const dlrm_bwd_timing* tm, hipStream_t st);
// bwd_tail.hip
int launch_segment_sort(const GroupArgs& g, hipStream_t st);
int launch_hot_rows(const GroupArgs& g, const UpdArgs& u, int G, int dtype, int opt, hipStream_t st);

}  // namespace dlrm
