// Backward grouping, steps 1-3: most-significant-digit partition of the (row, bag) pairs.
#include "bwd_common.h"

namespace dlrm {

// A bucket of n pairs goes to the list that the first workgroups of the reduce kernel take, if it is heavy.
__device__ inline void list_if_heavy(const GroupArgs& a, int k, int dg, uint32_t n) {
  if (n > a.big) a.over_list[atomicAdd(a.list_cnt, 1u)] = (uint32_t)((k << a.top_bits) + dg);
  if (n > (uint32_t)kBktCap) atomicAdd(a.over_cnt, 1u);
}

// --- 1. per-tile histogram of the partition digit ----------------------------------
// ITEMS positions per thread, as in the scatter.  While the row ids are on their way, the tile's first bag is
// searched for, so that the scatter starts from a record (TileRec).
template <typename IT, int ITEMS>
__global__ __launch_bounds__(kThreads) void bucket_hist_kernel(GroupArgs a) {
  __shared__ uint32_t h[kMaxBuckets];
  __shared__ uint32_t smem[kNW + 1];
  TileInfo ti;
  if (blockIdx.x == 0) {  // consumed by later launches of the same call
    for (int k = threadIdx.x; k < a.K; k += kThreads) a.hot_cnt[k] = 0u;
    if (threadIdx.x < 8) a.seg_meta[threadIdx.x] = 0u;
    if (threadIdx.x == 0) *a.over_cnt = *a.list_cnt = 0u;
  }
  if (!find_tile(a, blockIdx.x, ti, smem)) {
    if (threadIdx.x == 0) a.tile_rec[blockIdx.x].count = 0u;
    return;
  }
  const int nb = 1 << a.top_bits, tid = threadIdx.x;
  const IT* idx = static_cast<const IT*>(a.indices) + ti.start;
  const int shift = top_shift(a, ti.k);
  const uint32_t mask = (uint32_t)nb - 1;
  uint32_t key[ITEMS];
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const int i = j * kThreads + tid;
    key[j] = (uint32_t)idx[i < ti.count ? i : ti.count - 1];
  }
  for (int i = tid; i < nb; i += kThreads) h[i] = 0;
  __syncthreads();
  // the last bag b with off[b] <= P0, the tile's first position
  const int64_t* off = a.offsets + (int64_t)ti.k * (a.B + 1);
  const int64_t P0 = ti.start - ti.tbl_start;
  // (bags in unsigned 32 bits: a probe may end beyond 2^31)
  uint32_t lo = 0, hi = (uint32_t)a.B;  // off[lo] <= P0 (off[0] = 0); the answer lies in [lo, hi)
  while (hi - lo > 1u) {   // 256-ary search, uniform
    const uint32_t step = (hi - lo + kThreads - 1u) / kThreads;
    const uint32_t q = lo + (tid + 1u) * step;
    const int pred = (q < hi && off[q] <= P0) ? 1 : 0;
    const uint32_t cnt = (uint32_t)__syncthreads_count(pred);   // offsets are monotone: the first cnt probes pass
    const uint32_t nlo = lo + cnt * step;
    const uint32_t nhi = nlo + step < hi ? nlo + step : hi;
    lo = nlo;
    hi = nhi;
  }
#pragma unroll
  for (int j = 0; j < ITEMS; ++j)
    if (j * kThreads + tid < ti.count) atomicAdd(&h[(key[j] >> shift) & mask], 1u);
  __syncthreads();
  for (int i = tid; i < nb; i += kThreads) a.hist[(size_t)blockIdx.x * nb + i] = h[i];
  if (tid == 0)
    a.tile_rec[blockIdx.x] = TileRec{(uint32_t)ti.k, (uint32_t)ti.t, (uint32_t)ti.t0, (uint32_t)ti.nt, (uint32_t)ti.count,
                                     (uint32_t)ti.tbl_start, (uint32_t)shift, lo};
}

// --- 2. column scan (large batches only): counts -> pairs of the digit in earlier tiles ------
// hist[tile][digit] becomes the number of pairs of that digit in the table's earlier tiles, in
// place, and the digit's total goes to digit_total; the scatter turns totals into bucket starts
// itself.  A workgroup owns kScanDigits digits of one table and walks the table's tiles
// kScanSegs * kScanItems at a time: the loads of a round are in flight together, consecutive
// threads read consecutive digits of a tile.  Bound by the latency of a round (256 tiles).  The step
// it serves, before with one workgroup per table walking all of its (digit, tile) pairs / now:
// 4 tables of 164 K lookups 528 / 447 us, 64 tables of 524 K lookups 3016 / 2905 us, 8 tables of
// 103 K lookups with Adagrad 291 / 264 us.
constexpr int kScanDigits = 16, kScanSegs = kThreads / kScanDigits, kScanItems = 16;
__global__ __launch_bounds__(kThreads) void bucket_scan_kernel(GroupArgs a) {
  __shared__ uint32_t part[kScanSegs][kScanDigits];
  __shared__ uint32_t smem[kNW + 1];
  const int k = blockIdx.y, nb = 1 << a.top_bits;
  const int64_t tsize = (int64_t)1 << a.tile_shift;
  // first tile of table k = tiles of all earlier tables
  uint32_t mine = 0, t0;
  for (int j = threadIdx.x; j < k; j += kThreads)
    mine += (uint32_t)((a.tbl_off[j + 1] - a.tbl_off[j] + tsize - 1) >> a.tile_shift);
  block_exclusive_scan<kThreads>(mine, smem, &t0);
  const int nt = (int)((a.tbl_off[k + 1] - a.tbl_off[k] + tsize - 1) >> a.tile_shift);
  const int dl = threadIdx.x % kScanDigits, seg = threadIdx.x / kScanDigits;
  const int dg = blockIdx.x * kScanDigits + dl;
  uint32_t* col = a.hist + (size_t)t0 * nb + dg;
  uint32_t carry = 0;
  for (int r0 = 0; r0 < nt; r0 += kScanSegs * kScanItems) {   // uniform
    const int first = r0 + seg * kScanItems;
    uint32_t v[kScanItems], sum = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) v[j] = (dg < nb && first + j < nt) ? col[(size_t)(first + j) * nb] : 0u;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) sum += v[j];
    __syncthreads();   // the previous round's sums have been read
    part[seg][dl] = sum;
    __syncthreads();
    uint32_t run = carry;
#pragma unroll
    for (int s = 0; s < kScanSegs; ++s) {
      const uint32_t c = part[s][dl];
      run += s < seg ? c : 0u;
      carry += c;
    }
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
      if (dg < nb && first + j < nt) col[(size_t)(first + j) * nb] = run;
      run += v[j];
    }
  }
  if (seg == 0 && dg < nb && nt > 0) {
    a.digit_total[(size_t)k * nb + dg] = carry;
    list_if_heavy(a, k, dg, carry);
  }
}


// --- 3. stable scatter into buckets ---------------------------------------------------
// ITEMS positions per thread: the tile holds kThreads * ITEMS positions (GroupArgs::tile_shift agrees).  Bound by
// latency (a few workgroups per compute unit): all that the tile reads is requested at once, from one record.
// With the tile map, the search for the first bag, the bag starts and the row ids one after the other / now, kernel alone: 820
// tiles of 1024 15.9 / 14.0 us, 500 tiles 11.0 / 8.9 us (the histogram is no slower).
constexpr int kStartItems = 4;   // bag starts a thread looks at per round
template <typename IT, int ITEMS>
__global__ __launch_bounds__(kThreads) void bucket_scatter_kernel(GroupArgs a) {
  constexpr int TILE = kThreads * ITEMS;
  __shared__ uint32_t wcnt[kNW][kMaxBuckets];
  __shared__ uint32_t gofs[kMaxBuckets];
  __shared__ __align__(16) uint32_t skey[TILE];
  __shared__ __align__(16) uint32_t sval[TILE];
  __shared__ uint32_t smem[kNW + 1];
  const TileRec rec = a.tile_rec[blockIdx.x];
  if (rec.count == 0u) return;   // uniform
  TileInfo ti;
  ti.k = (int)rec.k;
  ti.t = (int)rec.t;
  ti.t0 = (int)rec.t0;
  ti.nt = (int)rec.nt;
  ti.count = (int)rec.count;
  ti.tbl_start = (int64_t)rec.tbl_start;
  ti.start = ti.tbl_start + ((int64_t)ti.t << a.tile_shift);
  const int nb = 1 << a.top_bits;
  const uint32_t mask = (uint32_t)nb - 1;
  const int lane = lane_id(), w = wave_id();
  const int tid = threadIdx.x;

  // ---- requested together: the tile's row ids (wave-striped), the starts of the bags behind its first one, and this
  // digit's counts in all tiles of the table
  const IT* kin = static_cast<const IT*>(a.indices) + ti.start;
  const int shift = (int)rec.shift;
  uint32_t key[ITEMS], val[ITEMS], dg[ITEMS], rnk[ITEMS];
  bool ok[ITEMS];
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const int li = w * (DLRM_WAVE * ITEMS) + j * DLRM_WAVE + lane;
    ok[j] = li < ti.count;
    key[j] = ok[j] ? (uint32_t)kin[li] : 0xFFFFFFFFu;
    dg[j] = (key[j] >> shift) & mask;
  }
  const int64_t* off = a.offsets + (int64_t)ti.k * (a.B + 1);
  const int64_t P0 = ti.start - ti.tbl_start;
  const uint32_t nbags = (uint32_t)a.B;   // (bags in unsigned 32 bits: a round may end beyond 2^31)
  const uint32_t b0 = rec.bag;
  int64_t starts[kStartItems];
#pragma unroll
  for (int q = 0; q < kStartItems; ++q) {
    const uint32_t b = b0 + 1u + q * kThreads + tid;
    starts[q] = off[b < nbags ? b : nbags];   // off[B]: the table's lookups, not before the tile's end
  }
  for (int i = tid; i < TILE; i += kThreads) skey[i] = 0;  // the bag-start counters
  // per digit: pairs of the digit in the table (stot) and in the table's earlier tiles (sbef)
  uint32_t* stot = &wcnt[0][0];
  uint32_t* sbef = &wcnt[1][0];
  if (a.fused_scan) {
    // Few tiles: every workgroup adds up the table's raw tile counts (a launch less).  nb / 4 threads
    // take 4 consecutive digits each; with fewer than 1024 digits up to kScanSegs times as many threads
    // split the tiles, so that 256 digits and 50 tiles are 13 dependent steps instead of 50.
    const int quads = nb >= 4 ? nb >> 2 : 1;
    const int segs = kThreads / quads < kScanSegs ? kThreads / quads : kScanSegs;
    const int quad = tid % quads, seg = tid / quads;
    const uint32_t* h0 = a.hist + (size_t)ti.t0 * nb;
    uint32_t tt[4] = {0, 0, 0, 0}, bb[4] = {0, 0, 0, 0};
    if (nb >= 4) {
      for (int t = seg < segs ? seg : ti.nt; t < ti.nt; t += segs * 8) {
        u32x4 c[8];
#pragma unroll
        for (int z = 0; z < 8; ++z) {
          const int tz = t + z * segs;
          c[z] = *reinterpret_cast<const u32x4*>(h0 + (size_t)(tz < ti.nt ? tz : ti.nt - 1) * nb + quad * 4);
        }
#pragma unroll
        for (int z = 0; z < 8; ++z) {
          const int tz = t + z * segs;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            tt[q] += tz < ti.nt ? c[z][q] : 0u;
            bb[q] += tz < ti.t ? c[z][q] : 0u;
          }
        }
      }
    } else {
      for (int t = seg < segs ? seg : ti.nt; t < ti.nt; t += segs) {
        for (int q = 0; q < nb; ++q) {
          const uint32_t c = h0[(size_t)t * nb + q];
          tt[q] += c;
          bb[q] += t < ti.t ? c : 0u;
        }
      }
    }
    if (seg < segs) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        stot[(seg * quads + quad) * 4 + q] = tt[q];   // segs * quads * 4 <= 1024 words
        sbef[(seg * quads + quad) * 4 + q] = bb[q];
      }
    }
  }
  // thread t owns the partition digits t*kDPT .. t*kDPT + kDPT-1
  uint32_t goff[kDPT], before[kDPT], total[kDPT];
  if (!a.fused_scan) {
#pragma unroll
    for (int q = 0; q < kDPT; ++q) {
      const int dgt = tid * kDPT + q;
      total[q] = dgt < nb ? a.digit_total[(size_t)ti.k * nb + dgt] : 0u;
      before[q] = dgt < nb ? a.hist[(size_t)blockIdx.x * nb + dgt] : 0u;
    }
  }
  __syncthreads();   // the counters are zero, the tile counts added up
  if (a.fused_scan) {
    const int row = nb >= 4 ? nb : 4, rows = kThreads * 4 / row < kScanSegs ? kThreads * 4 / row : kScanSegs;
#pragma unroll
    for (int q = 0; q < kDPT; ++q) {
      const int dgt = tid * kDPT + q;
      before[q] = total[q] = 0;
      if (dgt >= nb) continue;
      for (int sg = 0; sg < rows; ++sg) {
        total[q] += stot[sg * row + dgt];
        before[q] += sbef[sg * row + dgt];
      }
    }
  }

  // ---- bag of every position of the tile, from the starts of the bags that begin inside it, after P0
  for (uint32_t base = b0 + 1u;;) {
    int inside = 0;
#pragma unroll
    for (int q = 0; q < kStartItems; ++q) {
      const bool in = base + q * kThreads + tid < nbags && starts[q] < P0 + ti.count;
      if (in) atomicAdd(&skey[(int)(starts[q] - P0)], 1u);
      inside += in ? 1 : 0;
    }
    // monotone offsets: where a round has a bag beyond the tile, every later bag is
    if (__syncthreads_count(inside == kStartItems) < kThreads) break;
    base += kStartItems * kThreads;
#pragma unroll
    for (int q = 0; q < kStartItems; ++q) {
      const uint32_t b = base + q * kThreads + tid;
      starts[q] = off[b < nbags ? b : nbags];
    }
  }
  for (int i = tid; i < kNW * kMaxBuckets; i += kThreads) (&wcnt[0][0])[i] = 0;   // (the sums above have been read)
  {  // inclusive prefix of the start counters, thread t owning positions [t*ITEMS, (t+1)*ITEMS)
    uint32_t c[ITEMS], s = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; j += 4) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(skey + tid * ITEMS + j);
      c[j] = v.x;
      c[j + 1] = v.y;
      c[j + 2] = v.z;
      c[j + 3] = v.w;
      s += v.x + v.y + v.z + v.w;
    }
    uint32_t all;
    uint32_t run = b0 + block_exclusive_scan<kThreads>(s, smem, &all);
#pragma unroll
    for (int j = 0; j < ITEMS; j += 4) {
      u32x4 v;
      v.x = run + c[j];
      v.y = v.x + c[j + 1];
      v.z = v.y + c[j + 2];
      v.w = v.z + c[j + 3];
      run = v.w;
      *reinterpret_cast<u32x4*>(sval + tid * ITEMS + j) = v;
    }
  }
  __syncthreads();

  // ---- bags of this thread's (wave-striped) positions, then rank by partition digit
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const int li = w * (DLRM_WAVE * ITEMS) + j * DLRM_WAVE + lane;
    val[j] = ok[j] ? sval[li] : 0u;
    if (a.weights != nullptr && ok[j]) {  // uniform branch: weighted batch
      PosEntry pe;
      pe.bag = val[j];
      pe.w = a.weights[ti.start + li];
      a.pos_entry[ti.start + li] = pe;
      val[j] = (uint32_t)(P0 + li);       // position inside the table
    }
  }
  rank_items<ITEMS, kMaxBuckets>(dg, ok, a.top_bits, wcnt, rnk);
  __syncthreads();

  // ---- destination offsets of this tile's digits
  {
    uint32_t sum = 0, all;
#pragma unroll
    for (int q = 0; q < kDPT; ++q) sum += total[q];
    uint32_t base = block_exclusive_scan<kThreads>(sum, smem, &all);
#pragma unroll
    for (int q = 0; q < kDPT; ++q) {
      const int dgt = tid * kDPT + q;
      goff[q] = (uint32_t)ti.tbl_start + base + before[q];
      if (ti.t == 0 && dgt < nb) {
        a.bucket_start[(size_t)ti.k * nb + dgt] = (uint32_t)ti.tbl_start + base;
        if (a.fused_scan) list_if_heavy(a, ti.k, dgt, total[q]);
      }
      base += total[q];
    }
  }
  uint32_t lofs[kDPT], tot[kDPT];
  digit_offsets<kMaxBuckets>(nb, wcnt, smem, lofs, tot);
#pragma unroll
  for (int q = 0; q < kDPT; ++q) {
    const int dgt = tid * kDPT + q;
    if (dgt < nb) gofs[dgt] = goff[q] - lofs[q];
  }
  __syncthreads();

  // ---- stage in LDS in sorted order so that one digit's global writes are contiguous
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    if (ok[j]) {
      const uint32_t lp = wcnt[w][dg[j]] + rnk[j];
      skey[lp] = key[j];
      sval[lp] = val[j];
    }
  }
  __syncthreads();
  uint32_t* kout = a.keys[1];
  uint32_t* vout = a.vals[1];
  for (int lp = tid; lp < ti.count; lp += kThreads) {
    const uint32_t kk = skey[lp];
    const uint32_t dst = gofs[(kk >> shift) & mask] + (uint32_t)lp;
    kout[dst] = kk;
    vout[dst] = sval[lp];
  }
}


int enqueue_partition(const dlrm_sparse_batch* s, const GroupArgs& g, hipStream_t st) {
  const bool small = g.tile_shift == 10;
  if (g.idx32)
    hipLaunchKernelGGL((small ? bucket_hist_kernel<int32_t, kSmallItems> : bucket_hist_kernel<int32_t, kItems>), dim3(g.nt_max), dim3(kThreads), 0, st, g);
  else
    hipLaunchKernelGGL((small ? bucket_hist_kernel<int64_t, kSmallItems> : bucket_hist_kernel<int64_t, kItems>), dim3(g.nt_max), dim3(kThreads), 0, st, g);
  DLRM_CHECK_LAUNCH();
  if (!g.fused_scan) {
    hipLaunchKernelGGL(bucket_scan_kernel, dim3(div_up((int64_t)1 << g.top_bits, kScanDigits), s->K), dim3(kThreads), 0, st,
                       g);
    DLRM_CHECK_LAUNCH();
  }
  if (g.idx32) {
    if (small)
      hipLaunchKernelGGL((bucket_scatter_kernel<int32_t, kSmallItems>), dim3(g.nt_max), dim3(kThreads), 0, st, g);
    else
      hipLaunchKernelGGL((bucket_scatter_kernel<int32_t, kItems>), dim3(g.nt_max), dim3(kThreads), 0, st, g);
  } else {
    if (small)
      hipLaunchKernelGGL((bucket_scatter_kernel<int64_t, kSmallItems>), dim3(g.nt_max), dim3(kThreads), 0, st, g);
    else
      hipLaunchKernelGGL((bucket_scatter_kernel<int64_t, kItems>), dim3(g.nt_max), dim3(kThreads), 0, st, g);
  }
  DLRM_CHECK_LAUNCH();
  return DLRM_OK;
}

}  // namespace dlrm
