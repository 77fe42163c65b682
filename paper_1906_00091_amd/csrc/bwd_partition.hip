// Backward grouping, steps 1-3: most-significant-digit partition of the (row, bag) pairs.
#include "bwd_common.h"

namespace dlrm {

// A bucket of n pairs goes to the list that the first workgroups of the reduce kernel take, if it is heavy.
__device__ inline void list_if_heavy(const GroupArgs& a, int k, int dg, uint32_t n) {
  if (n > a.big) a.over_list[atomicAdd(a.list_cnt, 1u)] = (uint32_t)((k << a.top_bits) + dg);
  if (n > (uint32_t)kBktCap) atomicAdd(a.over_cnt, 1u);
}

// --- 1. per-tile histogram of the partition digit ----------------------------------
template <typename IT>
__global__ __launch_bounds__(kThreads) void bucket_hist_kernel(GroupArgs a) {
  __shared__ uint32_t h[kMaxBuckets];
  __shared__ uint32_t smem[kNW + 1];
  TileInfo ti;
  if (!find_tile(a, blockIdx.x, ti, smem)) return;
  const int nb = 1 << a.top_bits;
  for (int i = threadIdx.x; i < nb; i += kThreads) h[i] = 0;
  __syncthreads();
  const IT* idx = static_cast<const IT*>(a.indices) + ti.start;
  const int shift = top_shift(a, ti.k);
  const uint32_t mask = (uint32_t)nb - 1;
  for (int i = threadIdx.x; i < ti.count; i += kThreads)
    atomicAdd(&h[((uint32_t)idx[i] >> shift) & mask], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < nb; i += kThreads) a.hist[(size_t)blockIdx.x * nb + i] = h[i];
  if (blockIdx.x == 0 && threadIdx.x == 0) {  // consumed by later launches of the same call
    *a.over_cnt = 0u;
    *a.list_cnt = 0u;
    for (int k = 0; k < a.K; ++k) a.hot_cnt[k] = 0u;
    for (int i = 0; i < 8; ++i) a.seg_meta[i] = 0u;
  }
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
// ITEMS positions per thread: the tile holds kThreads * ITEMS positions (GroupArgs::tile_shift agrees)
template <typename IT, int ITEMS>
__global__ __launch_bounds__(kThreads) void bucket_scatter_kernel(GroupArgs a) {
  constexpr int TILE = kThreads * ITEMS;
  __shared__ uint32_t wcnt[kNW][kMaxBuckets];
  __shared__ uint32_t gofs[kMaxBuckets];
  __shared__ uint32_t skey[TILE];
  __shared__ uint32_t sval[TILE];
  __shared__ uint32_t smem[kNW + 1];
  __shared__ int sflag[1];
  TileInfo ti;
  if (!find_tile(a, blockIdx.x, ti, smem)) return;
  const int nb = 1 << a.top_bits;
  const uint32_t mask = (uint32_t)nb - 1;
  const int lane = lane_id(), w = wave_id();
  const int tid = threadIdx.x;

  // ---- requested first so that their latency hides behind the bag search: the tile's row ids
  // (wave-striped) and, for small batches, this digit's counts in all tiles of the table
  const IT* kin = static_cast<const IT*>(a.indices) + ti.start;
  const int shift = top_shift(a, ti.k);
  uint32_t key[ITEMS], val[ITEMS], dg[ITEMS], rnk[ITEMS];
  bool ok[ITEMS];
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const int li = w * (DLRM_WAVE * ITEMS) + j * DLRM_WAVE + lane;
    ok[j] = li < ti.count;
    key[j] = ok[j] ? (uint32_t)kin[li] : 0xFFFFFFFFu;
    dg[j] = (key[j] >> shift) & mask;
  }
  // per digit: pairs of the digit in the table (stot) and in the table's earlier tiles (sbef)
  uint32_t* stot = skey;
  uint32_t* sbef = sval;
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
  if (a.fused_scan) __syncthreads();
#pragma unroll
  for (int q = 0; q < kDPT; ++q) {
    const int dgt = tid * kDPT + q;
    before[q] = total[q] = 0;
    if (dgt >= nb) continue;
    if (a.fused_scan) {
      const int row = nb >= 4 ? nb : 4, rows = kThreads * 4 / row < kScanSegs ? kThreads * 4 / row : kScanSegs;
      for (int sg = 0; sg < rows; ++sg) {
        total[q] += stot[sg * row + dgt];
        before[q] += sbef[sg * row + dgt];
      }
    } else {
      total[q] = a.digit_total[(size_t)ti.k * nb + dgt];
      before[q] = a.hist[(size_t)blockIdx.x * nb + dgt];
    }
  }
  if (a.fused_scan) __syncthreads();   // skey and sval are written again below

  // ---- bag of every position of the tile, from the offsets
  // b0 = the bag holding the tile's first position: last b with off[b] <= P0.
  const int64_t* off = a.offsets + (int64_t)ti.k * (a.B + 1);
  const int64_t P0 = ti.start - ti.tbl_start;
  // (bags in unsigned 32 bits: a probe or a round may end beyond 2^31)
  const uint32_t nbags = (uint32_t)a.B;
  uint32_t lo = 0, hi = nbags;  // off[lo] <= P0 (off[0] = 0); the answer lies in [lo, hi)
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
  const uint32_t b0 = lo;
  for (int i = tid; i < TILE; i += kThreads) skey[i] = 0;  // skey doubles as the bag-start counters
  for (int i = tid; i < kNW * kMaxBuckets; i += kThreads) (&wcnt[0][0])[i] = 0;
  __syncthreads();
  for (uint32_t base = b0 + 1u;; base += kThreads) {  // bags that start inside the tile (after P0)
    const uint32_t b = base + tid;
    if (tid == 0) sflag[0] = (b >= nbags || off[b] >= P0 + ti.count) ? 1 : 0;
    if (b < nbags) {
      const int64_t ob = off[b];
      if (ob < P0 + ti.count) atomicAdd(&skey[(int)(ob - P0)], 1u);
    }
    __syncthreads();
    const int done = sflag[0];
    __syncthreads();
    // monotone offsets: once this round's first bag starts past the tile, every later one does;
    // a round whose first bag is inside may still have later bags inside, so go on
    if (done) break;
  }
  {  // inclusive prefix of the start counters, thread t owning positions [t*ITEMS, (t+1)*ITEMS)
    uint32_t c[ITEMS], s = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      c[j] = skey[tid * ITEMS + j];
      s += c[j];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan<kThreads>(s, smem, &total);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      run += c[j];
      sval[tid * ITEMS + j] = b0 + run;
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
  if (g.idx32)
    hipLaunchKernelGGL(bucket_hist_kernel<int32_t>, dim3(g.nt_max), dim3(kThreads), 0, st, g);
  else
    hipLaunchKernelGGL(bucket_hist_kernel<int64_t>, dim3(g.nt_max), dim3(kThreads), 0, st, g);
  DLRM_CHECK_LAUNCH();
  if (!g.fused_scan) {
    hipLaunchKernelGGL(bucket_scan_kernel, dim3(div_up((int64_t)1 << g.top_bits, kScanDigits), s->K), dim3(kThreads), 0, st,
                       g);
    DLRM_CHECK_LAUNCH();
  }
  const bool small = g.tile_shift == 10;
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
