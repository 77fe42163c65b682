// Backward tail: the segment sort (oversized lists the bucket kernel could not take) and the hot
// rows kernels.  A hot row is updated by the workgroup that completes its table; storage type and
// optimizer are run-time values there (a few rows per table).
#include "bwd_sort.h"

namespace dlrm {

// Every workgroup counts, per row of the segment, the pairs in the tiles before its own and in
// the whole segment (the segment's keys stream through L2), sorts its own tile in LDS, and
// writes each pair to  segment start + rows before + same row in earlier tiles + rank in tile:
// the segment ends up fully sorted by (row, position) in the other pair buffer.
__global__ __launch_bounds__(kThreads) void segment_sort_kernel(GroupArgs a) {
  __shared__ SortLds s;
  __shared__ uint32_t before[kSegKeys];
  __shared__ uint32_t base[kSegKeys];
  SegInfo sg;
  uint32_t t;
  // for the hot-row launch of this call (the reduce kernel has no register left for it: with this loop there the
  // fp32 Adagrad variant spilled, 13 tables of 37 K lookups 152 -> 158 us)
  if (blockIdx.x == 0)
    for (int k = threadIdx.x; k < a.K; k += kThreads) a.hot_done[k] = 0u;
  if (!find_segment_tile(a, &sg, &t)) return;
  const int tid = threadIdx.x;
  const uint32_t nkeys = 1u << sg.low_bits, mask = nkeys - 1u;
  const uint32_t tstart = t * kBktCap;
  const uint32_t cnt = sg.n - tstart < (uint32_t)kBktCap ? sg.n - tstart : (uint32_t)kBktCap;
  for (uint32_t i = tid; i < nkeys; i += kThreads) {
    before[i] = 0;
    base[i] = 0;
  }
  __syncthreads();
  const uint32_t* kin = a.keys[sg.src] + sg.start;
  for (uint32_t i0 = 0; i0 < sg.n; i0 += kThreads * 8) {  // 8 loads in flight per thread
    uint32_t kk[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t i = i0 + q * kThreads + tid;
      kk[q] = kin[i < sg.n ? i : sg.n - 1];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      // a wavefront covers 64 consecutive positions, all on one side of tstart (a multiple of 64).
      // Segments are dominated by a few rows: the lanes that agree with the first valid lane
      // are counted with ONE LDS atomic instead of a 64-way conflict on the same counter.
      const uint32_t i = i0 + q * kThreads + tid;
      const bool valid = i < sg.n;
      uint32_t* ctr = i < tstart ? before : base;
      const uint32_t r = kk[q] & mask;
      const unsigned long long vm = __ballot(valid);
      if (vm == 0ull) continue;  // wave-uniform
      const int first = __ffsll((long long)vm) - 1;
      const uint32_t r0 = __shfl(r, first, DLRM_WAVE);
      const unsigned long long same = __ballot(valid && r == r0);
      if (lane_id() == first) atomicAdd(&ctr[r0], (uint32_t)__popcll(same));
      if (valid && r != r0) atomicAdd(&ctr[r], 1u);
    }
  }
  __syncthreads();
  {  // base[r] <- number of pairs of the segment with a smaller row (exclusive scan of the totals)
    const uint32_t per = (nkeys + kThreads - 1) / kThreads;
    uint32_t sum = 0;
    for (uint32_t j = 0; j < per; ++j) {
      const uint32_t r = tid * per + j;
      if (r < nkeys) sum += before[r] + base[r];
    }
    uint32_t all;
    uint32_t run = block_exclusive_scan<kThreads>(sum, s.smem, &all);
    for (uint32_t j = 0; j < per; ++j) {
      const uint32_t r = tid * per + j;
      if (r < nkeys) {
        const uint32_t c = before[r] + base[r];
        base[r] = run;
        run += c;
      }
    }
  }
  __syncthreads();
  Bucket tb;
  tb.k = (int)sg.k;
  tb.start = sg.start + tstart;
  tb.n = cnt;
  tb.low_bits = (int)sg.low_bits;
  sort_bucket_lds(a, tb, s, (int)sg.src);
  uint32_t* kout = a.keys[sg.src ^ 1u] + sg.start;
  uint32_t* vout = a.vals[sg.src ^ 1u] + sg.start;
  for (uint32_t p = tid; p < cnt; p += kThreads) {
    const uint32_t key = s.skey[p];
    uint32_t lo = 0, hi = p;  // first position of this key in the sorted tile
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (s.skey[mid] < key) lo = mid + 1; else hi = mid;
    }
    const uint32_t r = key & mask;
    const uint32_t dst = base[r] + before[r] + (p - lo);
    kout[dst] = key;
    vout[dst] = s.sval[p];
  }
}


// --- the update of the hot rows -----------------------------------------------------------------
// The workgroup (bag group) of table k that leaves its partial sums last adds them up and updates the
// rows: a counter per table (zeroed by segment_sort_kernel of the same call) tells it so, and nobody waits.
// Every wavefront waits until its own partial sums have reached the L2 (a barrier alone does not wait for
// stores, and thread 0's write-back covers only what lies in the L2 by then); the barrier puts them before
// thread 0's release; its acquire and the second barrier put everybody's before the reads.  Uniform answer;
// all threads call it.
__device__ inline bool last_of_table(const GroupArgs& a, int k, uint32_t groups) {
  __shared__ uint32_t is_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    is_last = __hip_atomic_fetch_add(&a.hot_done[k], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == groups - 1u;
  __syncthreads();
  return is_last != 0u;
}

// A lane group of GL lanes (4 columns each) per hot run adds the run's partial sums in bag-group order
// and updates the row.
template <int DT, int OPT, int GL>
__device__ inline void finish_rows(const GroupArgs& a, const UpdArgs& u, int k, uint32_t base, uint32_t nruns, int groups) {
  const int chunk = threadIdx.x % GL;
  if (chunk * 4 >= u.d) return;
  char* W = static_cast<char*>(u.tables[k]);
  float* H = state_base<OPT>(u, k);
  for (uint32_t r = threadIdx.x / GL; r < nruns; r += kThreads / GL) {
    const float* part = a.huge_part + ((size_t)(base + r) * groups) * u.d + chunk * 4;
    const RowRef ref = row_ref<DT, OPT>(W, H, u.d, a.huge_runs[base + r].row, chunk);
    const RowVal val = row_load<DT, OPT>(ref);
    f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int g0 = 0; g0 < groups; g0 += 8) {
      f32x4 v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = loadf4(part + (size_t)(g0 + q < groups ? g0 + q : g0) * u.d);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (g0 + q < groups) sum += v[q];
    }
    row_update_store<DT, OPT>(ref, val, sum, u);
  }
}

// kind: storage type and optimizer of the call (row_kind), uniform
template <int GL>
__device__ inline void finish_table(const GroupArgs& a, const UpdArgs& u, int kind, int k, uint32_t base, uint32_t nruns,
                                    int groups) {
  if (!last_of_table(a, k, (uint32_t)groups)) return;
  switch (kind) {
    case DLRM_F32 * 2 + kSgd: finish_rows<DLRM_F32, kSgd, GL>(a, u, k, base, nruns, groups); break;
    case DLRM_F16 * 2 + kSgd: finish_rows<DLRM_F16, kSgd, GL>(a, u, k, base, nruns, groups); break;
    case DLRM_BF16 * 2 + kSgd: finish_rows<DLRM_BF16, kSgd, GL>(a, u, k, base, nruns, groups); break;
    case DLRM_F32 * 2 + kAdagrad: finish_rows<DLRM_F32, kAdagrad, GL>(a, u, k, base, nruns, groups); break;
    case DLRM_F16 * 2 + kAdagrad: finish_rows<DLRM_F16, kAdagrad, GL>(a, u, k, base, nruns, groups); break;
    case DLRM_BF16 * 2 + kAdagrad: finish_rows<DLRM_BF16, kAdagrad, GL>(a, u, k, base, nruns, groups); break;
  }
}

// start of table k's hot-run list, summed by a wavefront (hot_list_base walks the tables one by one)
__device__ inline uint32_t hot_list_base_wave(const GroupArgs& a, int k) {
  uint32_t base = 0;
  for (int j = lane_id(); j < k; j += DLRM_WAVE) base += (uint32_t)((a.tbl_off[j + 1] - a.tbl_off[j]) / kHugeRun) + 1u;
#pragma unroll
  for (int o = 1; o < DLRM_WAVE; o <<= 1) base += (uint32_t)__shfl_xor((int)base, o, DLRM_WAVE);
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
}

// First of the ascending bags list[0..n) at or after `bound`: seven probes a round are in flight
// together (a third of the dependent loads of a binary search).
__device__ inline uint32_t lower_bag(const uint32_t* list, uint32_t n, uint32_t bound) {
  uint32_t lo = 0, hi = n;
  while (lo < hi) {
    const uint32_t step = (hi - lo + 7u) >> 3;
    uint32_t probe[7], below = 0;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      const uint32_t q = lo + (uint32_t)(j + 1) * step - 1u;   // < n where it counts
      probe[j] = list[q < hi ? q : hi - 1u];
    }
#pragma unroll
    for (int j = 0; j < 7; ++j) below += (lo + (uint32_t)(j + 1) * step - 1u < hi && probe[j] < bound) ? 1u : 0u;
    // the first `below` probes lie before the answer, the next one (if there is one) does not
    const uint32_t end = lo + (below + 1u) * step - 1u;
    lo += below * step;
    if (below < 7u && end < hi) hi = end;
  }
  return lo;
}


// --- 5. hot rows: runs too long for one workgroup -------------------------------------------------
// A hot row is looked up by a large share of the bags.  Workgroup (g, k) takes bag group g of table k and
// adds, for each hot run of the table, the gradient rows of the run's entries whose bag lies in the
// group; partial sums per (run, bag group) go to global memory, and finish_table adds them in group order.
// A run's bags ascend, so a search gives its first entry of a group.  Three ways to sum, all in an order
// fixed by the batch:
//   weighted batches     : bag tiles of gradient rows staged in LDS (hot_rows_weighted_kernel),
//   fewer than kDenseFrom hot rows in the table : gathered bag by bag (sum_few_runs),
//   more                 : a dense contraction on the matrix cores (hot_rows_dense_kernel).

// Entry e + slot of the 64 values the lanes hold in `v` (e: uniform).  Few slots: scalar lane
// reads and selects, no LDS round trip; many slots: a lane permute.
template <int S>
__device__ inline uint32_t lane_entry(uint32_t v, uint32_t e, int slot) {
  if constexpr (S <= 4) {
    uint32_t r = (uint32_t)__builtin_amdgcn_readlane((int)v, (int)(e & 63u));
#pragma unroll
    for (int sl = 1; sl < S; ++sl) {
      const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)v, (int)((e + sl) & 63u));
      r = slot == sl ? o : r;
    }
    return r;
  } else {
    return (uint32_t)__shfl((int)v, (int)((e + (uint32_t)slot) & 63u), DLRM_WAVE);
  }
}

// Weighted batches.  The next tile travels in registers while the current one is consumed; every
// wavefront adds the rows of its runs' entries from LDS, each times the entry's weight.
template <int G>
__global__ __launch_bounds__(kThreads) void hot_rows_weighted_kernel(GroupArgs a, UpdArgs u, int kind, int ngroups,
                                                                     int ntiles) {
  constexpr int S = DLRM_WAVE / G;
  constexpr int MR = kHotRunsPerWave;
  constexpr int NT = kHotTilesPerGroup;
  constexpr int HU = S <= 8 ? 8 : DLRM_WAVE / S;  // HU * S entries per round, never past the 64 held
  constexpr int NG = kThreads / G;                // gradient rows staged per pass of the workgroup
  constexpr int NP = kHotStagePasses;
  constexpr int TB = NG * NP;                     // bags per tile: TB * d <= kHotTileFloats
  const uint32_t GB = (uint32_t)(TB * ntiles);    // bags per workgroup, ntiles <= NT
  __shared__ float tile[kHotTileFloats + kHotZeroRow];  // gradient rows of a bag tile, then a row of zeros
  __shared__ uint32_t cursor[kNW * MR][NT + 1];  // first entry of a run at or after every tile boundary
  __shared__ uint32_t rsrc[kNW * MR];            // pair buffer holding the run
  // a run lists positions; bag and weight are looked up by position
  const int64_t tbl = a.tbl_off[blockIdx.y];
  const int k = blockIdx.y, g = blockIdx.x;
  const uint32_t nruns = a.hot_cnt[k];
  if (nruns == 0) return;  // uniform
  const uint32_t base = hot_list_base_wave(a, k);
  const int lane = lane_id(), w = wave_id(), tid = threadIdx.x;
  const int slot = lane / G, chunk = lane % G;
  const int grp = tid / G;
  const bool col_ok = chunk * 4 < u.d;
  const int cchunk = col_ok ? chunk : 0;  // lanes past the last column shadow column group 0, never store
  // unsigned: the last group may end beyond 2^31
  const uint32_t bag_lo = (uint32_t)g * GB;
  const uint32_t bag_hi = bag_lo + GB < (uint32_t)a.B ? bag_lo + GB : (uint32_t)a.B;
  const float* gk = u.dS + (int64_t)k * u.stride_k + cchunk * 4;
  for (int i = tid; i < kHotZeroRow; i += kThreads) tile[kHotTileFloats + i] = 0.0f;
  for (uint32_t r0 = 0; r0 < nruns; r0 += kNW * MR) {  // uniform
    __syncthreads();
    for (int task = tid; task < kNW * MR * (ntiles + 1); task += kThreads) {
      const int rl = task / (ntiles + 1), tb = task - rl * (ntiles + 1);
      const uint32_t r = r0 + (uint32_t)rl;
      uint32_t c = 0;
      if (r < nruns) {
        const HugeRun hr = a.huge_runs[base + r];
        const uint32_t* bags = (hr.src ? a.vals[1] : a.vals[0]) + hr.start;
        const uint32_t bnd = bag_lo + (uint32_t)(tb * TB);
        const uint32_t bound = bnd < bag_hi ? bnd : bag_hi;
        uint32_t lo = 0, hi = hr.len;
        while (lo < hi) {
          const uint32_t mid = (lo + hi) >> 1;
          if (a.pos_entry[tbl + bags[mid]].bag < bound) lo = mid + 1; else hi = mid;
        }
        c = hr.start + lo;
        if (tb == 0) rsrc[rl] = hr.src;
      }
      cursor[rl][tb] = c;
    }
    __syncthreads();
    const uint32_t* bags[MR];
    f32x4 acc[MR];
#pragma unroll
    for (int i = 0; i < MR; ++i) {
      const int rl = w + kNW * i;
      acc[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      bags[i] = (r0 + (uint32_t)rl < nruns && rsrc[rl]) ? a.vals[1] : a.vals[0];
    }
    // staging registers: row p*NG + grp of a tile, this lane's 4 columns (rows past the tile's
    // end repeat its last row and are never stored)
    f32x4 stage[NP];
    {
      const int nb = bag_hi - bag_lo < (uint32_t)TB ? (int)(bag_hi - bag_lo) : TB;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int bb = p * NG + grp < nb ? p * NG + grp : nb - 1;
        stage[p] = loadf4(gk + (int64_t)(bag_lo + bb) * u.stride_b);
      }
    }
    int t = 0;
    for (uint32_t tb0 = bag_lo; tb0 < bag_hi; tb0 += TB, ++t) {  // uniform
      const int nb = bag_hi - tb0 < (uint32_t)TB ? (int)(bag_hi - tb0) : TB;
      // the first 64 bags of every run of this wave are requested before the tile is stored
      uint32_t first[MR];
#pragma unroll
      for (int i = 0; i < MR; ++i) {
        const uint32_t c0 = cursor[w + kNW * i][t], c1 = cursor[w + kNW * i][t + 1];
        first[i] = 0;
        if (c0 + (uint32_t)lane < c1) first[i] = bags[i][c0 + lane];
      }
      __syncthreads();  // the previous tile has been consumed
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int bb = p * NG + grp;
        if (bb < nb && col_ok) storef4(tile + bb * u.d + chunk * 4, stage[p]);
      }
      __syncthreads();
      if (tb0 + TB < bag_hi) {  // uniform: the next tile travels while this one is summed
        const int nn = bag_hi - (tb0 + TB) < (uint32_t)TB ? (int)(bag_hi - (tb0 + TB)) : TB;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          const int bb = p * NG + grp < nn ? p * NG + grp : nn - 1;
          stage[p] = loadf4(gk + (int64_t)(tb0 + TB + bb) * u.stride_b);
        }
      }
#pragma unroll
      for (int i = 0; i < MR; ++i) {
        // the cursors are the same in every lane: scalar loop control
        const uint32_t c0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cursor[w + kNW * i][t]);
        const uint32_t c1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cursor[w + kNW * i][t + 1]);
        uint32_t cur = first[i];
        for (uint32_t e0 = c0; e0 < c1; e0 += DLRM_WAVE) {
          uint32_t nxt = 0;  // the next 64 bags travel while these are summed
          if (e0 + DLRM_WAVE + (uint32_t)lane < c1) nxt = bags[i][e0 + DLRM_WAVE + lane];
          const uint32_t cnt = c1 - e0 < (uint32_t)DLRM_WAVE ? c1 - e0 : (uint32_t)DLRM_WAVE;
          // every entry on its own: LDS offset of its bag's gradient row and its weight
          uint32_t moff = (uint32_t)kHotTileFloats;  // entries past the end: the row of zeros, weight 0
          float mw = 0.0f;
          if ((uint32_t)lane < cnt) {
            const PosEntry pe = a.pos_entry[tbl + cur];
            moff = (pe.bag - tb0) * (uint32_t)u.d;
            mw = pe.w;
          }
          for (uint32_t e = 0; e < cnt; e += HU * S) {
            f32x4 v[HU];
            float m[HU];
#pragma unroll
            for (int q = 0; q < HU; ++q) {
              v[q] = loadf4(tile + lane_entry<S>(moff, e + (uint32_t)(q * S), slot) + cchunk * 4);
              m[q] = u2f(lane_entry<S>(f2u(mw), e + (uint32_t)(q * S), slot));
            }
#pragma unroll
            for (int q = 0; q < HU; ++q) {
              acc[i].x = fmaf(m[q], v[q].x, acc[i].x);
              acc[i].y = fmaf(m[q], v[q].y, acc[i].y);
              acc[i].z = fmaf(m[q], v[q].z, acc[i].z);
              acc[i].w = fmaf(m[q], v[q].w, acc[i].w);
            }
          }
          cur = nxt;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < MR; ++i) {
      const uint32_t r = r0 + w + kNW * i;
      if (r >= nruns) continue;  // wave-uniform
      f32x4 tot = acc[i];
#pragma unroll
      for (int o = G; o < DLRM_WAVE; o <<= 1) {
        tot.x += __shfl_xor(tot.x, o, DLRM_WAVE);
        tot.y += __shfl_xor(tot.y, o, DLRM_WAVE);
        tot.z += __shfl_xor(tot.z, o, DLRM_WAVE);
        tot.w += __shfl_xor(tot.w, o, DLRM_WAVE);
      }
      float* part = a.huge_part + ((size_t)(base + r) * ngroups) * u.d;
      if (slot == 0 && col_ok) storef4(part + (size_t)g * u.d + chunk * 4, tot);
    }
  }
  finish_table<G>(a, u, kind, k, base, nruns, ngroups);
}


// Few hot rows: the four wavefronts of the workgroup own a quarter of its bags each and gather every
// distinct bag's gradient row of every run once (neighbouring entries of one bag are folded into a
// multiplicity), U * 4 bags at a time; the wavefronts' sums are added in bag order.  Bound by the chain
// search -> entries -> rows, so what counts is many wavefronts with few bags each (see hot_bag_groups):
// with groups of 2048 bags as before and LDS tiles, 26 bf16 tables of up to 10 M rows, 1.06 M lookups,
// 49 hot rows took 81 us, now 18 us with the rows updated (and the launch that did so gone).
template <int NH>
__device__ inline void sum_few_runs(const GroupArgs& a, const UpdArgs& u, int k, int g, uint32_t base, uint32_t nruns,
                                    int ngroups, uint32_t wb_lo, uint32_t wb_hi, uint32_t* lds) {
  constexpr int U = NH == 1 ? 8 : NH == 2 ? 4 : 2;
  const int lane = lane_id(), w = wave_id();
  const int m = lane & 15, kk = lane >> 4;
  const unsigned long long lt = (1ull << lane) - 1ull;
  const float* gk = u.dS + (int64_t)k * u.stride_k + 4 * m;
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  float* red = reinterpret_cast<float*>(lds);               // [wavefront][run][d]
  uint32_t* fold = lds + kNW * (kDenseFrom - 1) * 64 * NH + w * 2 * DLRM_WAVE;   // this wavefront's bags and multiplicities
  // lane r keeps run r's state; every run's first 64 entries are requested together
  uint32_t pos = 0, end = 0, src = 0;
  if ((uint32_t)lane < nruns && wb_lo < wb_hi) {
    const HugeRun hr = a.huge_runs[base + (uint32_t)lane];
    pos = hr.start + lower_bag((hr.src ? a.vals[1] : a.vals[0]) + hr.start, hr.len, wb_lo);
    end = hr.start + hr.len;
    src = hr.src;
  }
  uint32_t ent[kDenseFrom - 1];
#pragma unroll
  for (int q = 0; q < kDenseFrom - 1; ++q) {
    const uint32_t pq = (uint32_t)__builtin_amdgcn_readlane((int)pos, q);
    const uint32_t eq = (uint32_t)__builtin_amdgcn_readlane((int)end, q);
    const uint32_t* lq = __builtin_amdgcn_readlane((int)src, q) ? a.vals[1] : a.vals[0];
    ent[q] = 0xFFFFFFFFu;
    if (pq + (uint32_t)lane < eq) ent[q] = lq[pq + (uint32_t)lane];
  }
#pragma unroll
  for (int q = 0; q < kDenseFrom - 1; ++q) {
    if ((uint32_t)q >= nruns) continue;  // uniform
    uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)pos, q);
    const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)end, q);
    const uint32_t* lq = __builtin_amdgcn_readlane((int)src, q) ? a.vals[1] : a.vals[0];
    f32x4 acc[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) acc[h] = zero;
    uint32_t cur = ent[q];   // past the run's end: no bag
    for (;;) {
      const unsigned long long in = __ballot(cur < wb_hi);   // ascending: a prefix of the lanes
      const uint32_t cnt = (uint32_t)__popcll(in);
      if (cnt == 0u) break;  // wave-uniform
      const bool more = cnt == (uint32_t)DLRM_WAVE && c + (uint32_t)DLRM_WAVE < e;
      uint32_t nxt = 0xFFFFFFFFu;
      c += DLRM_WAVE;
      if (more && c + (uint32_t)lane < e) nxt = lq[c + (uint32_t)lane];
      // the first entry of each distinct bag carries how many follow
      const uint32_t prev = (uint32_t)__shfl_up((int)cur, 1, DLRM_WAVE);
      const bool head = (uint32_t)lane < cnt && (lane == 0 || cur != prev);
      const unsigned long long hm = __ballot(head);
      const uint32_t nh = (uint32_t)__popcll(hm);
      const unsigned long long rest = (hm >> lane) >> 1;
      const uint32_t nextp = rest ? (uint32_t)lane + (uint32_t)__ffsll((long long)rest) : cnt;
      if (head) {
        fold[__popcll(hm & lt)] = cur;
        fold[DLRM_WAVE + __popcll(hm & lt)] = nextp - (uint32_t)lane;
      }
      for (uint32_t i0 = 0; i0 < nh; i0 += U * 4) {   // wave-uniform
        f32x4 v[U][NH];
        float mult[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const uint32_t i = i0 + (uint32_t)(j * 4 + kk);
          const uint32_t bag = fold[i < nh ? i : nh - 1u];
          mult[j] = (float)fold[DLRM_WAVE + (i < nh ? i : nh - 1u)];
          const float* row = gk + (int64_t)bag * u.stride_b;
#pragma unroll
          for (int h = 0; h < NH; ++h) v[j][h] = loadf4(row + (64 * h + 4 * m < u.d ? 64 * h : -4 * m));
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
          if (i0 + (uint32_t)(j * 4 + kk) < nh) {
#pragma unroll
            for (int h = 0; h < NH; ++h) {
              acc[h].x = fmaf(mult[j], v[j][h].x, acc[h].x);
              acc[h].y = fmaf(mult[j], v[j][h].y, acc[h].y);
              acc[h].z = fmaf(mult[j], v[j][h].z, acc[h].z);
              acc[h].w = fmaf(mult[j], v[j][h].w, acc[h].w);
            }
          }
        }
      }
      if (!more) break;  // wave-uniform
      cur = nxt;
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) {
#pragma unroll
      for (int o = 16; o < DLRM_WAVE; o <<= 1) {
        acc[h].x += __shfl_xor(acc[h].x, o, DLRM_WAVE);
        acc[h].y += __shfl_xor(acc[h].y, o, DLRM_WAVE);
        acc[h].z += __shfl_xor(acc[h].z, o, DLRM_WAVE);
        acc[h].w += __shfl_xor(acc[h].w, o, DLRM_WAVE);
      }
      if (kk == 0 && 64 * h + 4 * m < u.d) storef4(red + (w * (kDenseFrom - 1) + q) * u.d + 64 * h + 4 * m, acc[h]);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x * 4; i < (int)nruns * u.d; i += kThreads * 4) {   // d is a multiple of 4
    const int q = i / u.d, col = i - q * u.d;
    f32x4 sum = loadf4(red + q * u.d + col);
#pragma unroll
    for (int x = 1; x < kNW; ++x) sum += loadf4(red + (x * (kDenseFrom - 1) + q) * u.d + col);
    storef4(a.huge_part + ((size_t)(base + q) * ngroups + g) * u.d + col, sum);
  }
}


// --- 5b. many hot rows in one table: the same pass as a dense product on the matrix cores -----------
// With many hot rows per table (a skewed table: the hottest few are in nearly every bag) a gradient row
// would be read once per (hot row, bag) that meets.  Here the multiplicities of kDenseRuns hot rows against a tile of bags are
// first counted into a small matrix C[run][bag] in LDS (integer atomics: exact, order-free); then
// G_hot[run][col] += sum_bag C[run][bag] * dS[bag][col] is a dense contraction over the bags of the
// tile, done with v_mfma_f32_16x16x4_f32: runs are the M index (two blocks of 16), four bags per
// instruction.
//
// Every wavefront works alone: it owns a quarter of the workgroup's bags, its own count matrix and
// accumulators for all runs and columns, and takes its gradient rows straight from global memory,
// so there is no barrier anywhere in the streaming loop and wavefronts in different phases
// (list reads, counting, contraction) fill each other's gaps.  The four partial results are added
// in bag order at the end.
//   16x16x4 layout: lane l supplies A[m = l%16][k = l/16] and B[k = l/16][n = l%16] and holds
//   D[m = 4*(l/16) + v][n = l%16] in element v of its accumulator.
//   Which column the N index n stands for is free as long as B and D agree: lane l loads the 16 bytes
//   dS[bag k][64h + 4n .. 64h + 4n + 3] with one instruction (a bag row is read as contiguous 256-byte
//   pieces) and component c of that load is the B operand of contraction (h, c), whose result
//   column n is gradient column 64h + 4n + c.
// A count of zero still multiplies the bag's gradient: a non-finite gradient entry of a bag reaches
// every hot row of this pass, not only the rows the bag looked up.
constexpr int kDenseRuns = 32;      // hot rows per pass of a workgroup
constexpr int kDenseTile = 64;      // bags per tile of a wavefront
constexpr int kDenseCStride = 68;   // words per run of the count matrix: 4m + k is a different bank for all 64 lanes
constexpr int kDensePre = 4;        // 4-bag steps of gradient rows in flight
constexpr int kDenseHeavy = 4;      // the longest runs of a pass: 256 list entries per request instead of 64

// Bag groups of an unweighted batch: as many as fill the machine once (gfx950: 256 compute units, three resident
// workgroups each, two for rows above 128 columns) with the tables that do have hot rows, which only the device knows;
// a wavefront's quarter of a group is whole tiles.  With the groups that fill it if every table has hot rows, one table
// of 3 hot rows (20 lookups a bag, batch 16384, d = 64) among 300 / 800 / 2000 (batch 8192) tables: update
// 1346 / 3098 / 3047 us; with these: 671 / 1624 / 2258 us; one such table among 26, batch 65536: 398 and 311 us; every
// table such a one, one lookup a bag, 100 tables: 182 and 184 us.
constexpr int hot_slots(int nh) { return 256 * (nh <= 2 ? 3 : 2); }
constexpr int kHotUnit = kNW * kDenseTile;
constexpr int kHotGroupMin = 512;   // bags of a group that more workgroups than all tables' share may be launched for

template <int NH>   // 64-column pieces of a gradient row
__global__ __launch_bounds__(kThreads, NH <= 2 ? 3 : 2) void hot_rows_dense_kernel(GroupArgs a, UpdArgs u, int kind) {
  constexpr int R = kDenseRuns, TB = kDenseTile, CS = kDenseCStride, PRE = NH <= 2 ? kDensePre : kDensePre / 2;
  static_assert(R * CS * kNW >= R * 64 * NH, "the reduction buffer aliases the count matrices");
  static_assert(R * CS * kNW >= kNW * (kDenseFrom - 1) * 64 * NH + kNW * 2 * DLRM_WAVE, "and so do sum_few_runs' buffers");
  __shared__ __align__(16) uint32_t cmat[kNW][R * CS];   // per wavefront: multiplicity of run r in bag tb0 + b at [r * CS + b]
  const uint32_t hot_tables = a.seg_meta[kHotTables];
  if (hot_tables == 0u) return;  // uniform, as is all up to the bags
  uint32_t want = (uint32_t)hot_slots(NH) / hot_tables;
  want = want < gridDim.x ? (want > 1u ? want : 1u) : gridDim.x;
  // (unsigned: the last group may end beyond 2^31)
  const uint32_t nbags = (uint32_t)a.B;
  const uint32_t group_bags = ((nbags + want - 1u) / want + (uint32_t)kHotUnit - 1u) / (uint32_t)kHotUnit * (uint32_t)kHotUnit;
  const int ngroups = (int)((nbags + group_bags - 1u) / group_bags);   // <= want
  // the first K * ngroups workgroups in launch order are the ones at work: neighbours go to different dies, whereas
  // the first ngroups of every gridDim.x may all go to one
  const int64_t id = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (id >= (int64_t)a.K * ngroups) return;
  const int k = (int)(id / ngroups), g = (int)(id - (int64_t)k * ngroups);
  const uint32_t nruns = a.hot_cnt[k];
  if (nruns == 0u) return;
  const uint32_t base = hot_list_base_wave(a, k);
  const int lane = lane_id(), w = wave_id();
  const int m = lane & 15, kk = lane >> 4;
  // this wavefront's bags
  const uint32_t quarter = group_bags / kNW;
  uint32_t wb_lo = (uint32_t)g * group_bags + (uint32_t)w * quarter;
  wb_lo = wb_lo < nbags ? wb_lo : nbags;
  const uint32_t wb_hi = wb_lo + quarter < nbags ? wb_lo + quarter : nbags;
  if (nruns < (uint32_t)kDenseFrom) {  // uniform
    sum_few_runs<NH>(a, u, k, g, base, nruns, ngroups, wb_lo, wb_hi, &cmat[0][0]);
    finish_table<16 * NH>(a, u, kind, k, base, nruns, ngroups);
    return;
  }
  const float* gk = u.dS + (int64_t)k * u.stride_k;
  // lanes whose columns lie past the row's end load its first four columns (no branch around a load; the
  // addresses right behind the last row of dS may not be mapped) and never store
  bool col_ok[NH];
  int hoff[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    col_ok[h] = 64 * h + 4 * m < u.d;
    hoff[h] = col_ok[h] ? 64 * h + 4 * m : 0;
  }
  uint32_t* cm = cmat[w];
  float* red = reinterpret_cast<float*>(&cmat[0][0]);
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  for (uint32_t r0 = 0; r0 < nruns; r0 += R) {  // uniform
    // lane r keeps the state of one run of this pass: next entry for this wavefront's bags (a binary
    // search: a run's bags ascend), end of the run, pair buffer that holds it.  The runs are dealt to
    // the lanes by length, longest first: the first kDenseHeavy get the wide list requests.
    uint32_t pos = 0, end = 0, src = 0, ridx = 0xFFFFFFFFu;
    {
      uint32_t len = 0;
      HugeRun hr;
      hr.start = hr.len = hr.src = 0;
      if (lane < R && r0 + (uint32_t)lane < nruns) {
        hr = a.huge_runs[base + r0 + (uint32_t)lane];
        len = hr.len;
      }
      uint32_t rank = 0;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uint32_t lj = (uint32_t)__builtin_amdgcn_readlane((int)len, j);
        rank += (lj > len || (lj == len && j < lane)) ? 1u : 0u;
      }
      rank = lane < R ? rank : (uint32_t)lane;
      uint32_t lo = 0;
      if (len != 0 && wb_lo < wb_hi) {
        lo = lower_bag((hr.src ? a.vals[1] : a.vals[0]) + hr.start, hr.len, wb_lo);
      }
      const bool live = len != 0 && wb_lo < wb_hi;
      pos = (uint32_t)__builtin_amdgcn_ds_permute((int)(rank * 4), (int)(live ? hr.start + lo : 0u));
      end = (uint32_t)__builtin_amdgcn_ds_permute((int)(rank * 4), (int)(live ? hr.start + hr.len : 0u));
      src = (uint32_t)__builtin_amdgcn_ds_permute((int)(rank * 4), (int)hr.src);
      ridx = (uint32_t)__builtin_amdgcn_ds_permute((int)(rank * 4), (int)(len != 0 ? r0 + (uint32_t)lane : 0xFFFFFFFFu));
    }
    const int nr = nruns - r0 < (uint32_t)R ? (int)(nruns - r0) : R;  // uniform; the absent runs are the last lanes
    f32x4 acc[2][NH][4];   // [run block][column piece][component of the 16-byte load]
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[0][h][c] = acc[1][h][c] = zero;
#pragma unroll 1
    for (uint32_t tb0 = wb_lo; tb0 < wb_hi; tb0 += TB) {  // wave-uniform
      const uint32_t bound = wb_hi - tb0 < (uint32_t)TB ? wb_hi : tb0 + TB;
      f32x4 bq[PRE][NH];
      for (int i = lane; i < R * CS / 4; i += DLRM_WAVE) reinterpret_cast<u32x4*>(cm)[i] = u32x4{0u, 0u, 0u, 0u};
      // count: the entries of every run that fall into this tile are a prefix of what is left of it
      {
        constexpr int HV = kDenseHeavy;
        // every run's request goes out before the first answer is used: 256 entries of each of the
        // longest runs, 64 of the others (requests past a run's end repeat its last entry and are
        // masked afterwards; an absent run has pos = end = 0)
        u32x4 hent[HV];
        uint32_t ent[R - HV];
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const uint32_t pq = (uint32_t)__builtin_amdgcn_readlane((int)pos, q);
          const uint32_t eq = (uint32_t)__builtin_amdgcn_readlane((int)end, q);
          const uint32_t* lq = __builtin_amdgcn_readlane((int)src, q) ? a.vals[1] : a.vals[0];
          const uint32_t last = eq ? eq - 1u : 0u;
          if (q < HV) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const uint32_t x = pq + (uint32_t)(4 * lane + t);
              hent[q < HV ? q : 0][t] = lq[x < last ? x : last];
            }
          } else {
            const uint32_t x = pq + (uint32_t)lane;
            ent[q >= HV ? q - HV : 0] = lq[x < last ? x : last];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < R; ++q) {
          if (q == R / 2) {
            // the first gradient rows travel while the second half of the runs is counted (bags past
            // the end repeat the last one; their counts stay zero)
#pragma unroll
            for (int s = 0; s < PRE; ++s) {
              const uint32_t bag = tb0 + 4 * s + kk < wb_hi ? tb0 + 4 * s + kk : wb_hi - 1u;
#pragma unroll
              for (int h = 0; h < NH; ++h) bq[s][h] = loadf4(gk + (int64_t)bag * u.stride_b + hoff[h]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          if (q >= nr) continue;  // uniform (the gradient requests above are not skipped)
          uint32_t pq = (uint32_t)__builtin_amdgcn_readlane((int)pos, q);
          const uint32_t eq = (uint32_t)__builtin_amdgcn_readlane((int)end, q);
          uint32_t* crow = cm + q * CS - tb0;
          uint32_t n = 0, full;
          if (q < HV) {
            full = 4u * DLRM_WAVE;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const uint32_t x = pq + (uint32_t)(4 * lane + t);
              const uint32_t bag = hent[q < HV ? q : 0][t];
              const bool in = x < eq && bag < bound;
              if (in) atomicAdd(crow + bag, 1u);
              n += (uint32_t)__popcll(__ballot(in));
            }
          } else {
            full = (uint32_t)DLRM_WAVE;
            const uint32_t x = pq + (uint32_t)lane;
            const uint32_t bag = ent[q >= HV ? q - HV : 0];
            const bool in = x < eq && bag < bound;
            if (in) atomicAdd(crow + bag, 1u);
            n = (uint32_t)__popcll(__ballot(in));
          }
          pq += n;
          while (n == full) {   // wave-uniform: every requested entry was inside the tile
            const uint32_t* lq = __builtin_amdgcn_readlane((int)src, q) ? a.vals[1] : a.vals[0];
            full = 4u * DLRM_WAVE;
            uint32_t bag[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const uint32_t x = pq + (uint32_t)(t * DLRM_WAVE + lane);
              bag[t] = 0xFFFFFFFFu;
              if (x < eq) bag[t] = lq[x];
            }
            n = 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {   // ascending bags: those inside are a prefix
              const bool in = bag[t] < bound;
              if (in) atomicAdd(crow + bag[t], 1u);
              n += (uint32_t)__popcll(__ballot(in));
            }
            pq += n;
          }
          pos = lane == q ? pq : pos;
        }
      }
      // contract over the bags of the tile, four per step
#pragma unroll
      for (int s = 0; s < TB / 4; ++s) {
        const float a0 = (float)cm[m * CS + 4 * s + kk];
        const float a1 = (float)cm[(16 + m) * CS + 4 * s + kk];
        f32x4 cur[NH];
#pragma unroll
        for (int h = 0; h < NH; ++h) cur[h] = bq[s % PRE][h];
        if (s + PRE < TB / 4) {
          const uint32_t bag = tb0 + 4 * (s + PRE) + kk < wb_hi ? tb0 + 4 * (s + PRE) + kk : wb_hi - 1u;
#pragma unroll
          for (int h = 0; h < NH; ++h) bq[s % PRE][h] = loadf4(gk + (int64_t)bag * u.stride_b + hoff[h]);
        }
        __builtin_amdgcn_sched_barrier(0);   // the request stays PRE steps ahead of its use
#pragma unroll
        for (int h = 0; h < NH; ++h) {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            acc[0][h][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, cur[h][c], acc[0][h][c], 0, 0, 0);
            acc[1][h][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, cur[h][c], acc[1][h][c], 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // the four wavefronts' results added in bag order: wavefront 0 takes in 1, 2, 3 through LDS
    // (run slot r, column j at red[r * d + j]).  out[mb][h][v]: run slot 16*mb + 4*(l/16) + v, the four
    // columns 64h + 4*(l%16) + c.
    f32x4 out[2][NH][4];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          out[mb][h][v] = f32x4{acc[mb][h][0][v], acc[mb][h][1][v], acc[mb][h][2][v], acc[mb][h][3][v]};
    __syncthreads();   // every count matrix has been consumed
    for (int from = 1; from < kNW; ++from) {  // uniform
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (w == from && col_ok[h]) storef4(red + (mb * 16 + kk * 4 + v) * u.d + 64 * h + 4 * m, out[mb][h][v]);
      __syncthreads();
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (w == 0 && col_ok[h]) out[mb][h][v] += loadf4(red + (mb * 16 + kk * 4 + v) * u.d + 64 * h + 4 * m);
      __syncthreads();
    }
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        // the run that was dealt to accumulator row mb*16 + kk*4 + v
        const uint32_t run = (uint32_t)__shfl((int)ridx, mb * 16 + kk * 4 + v, DLRM_WAVE);
#pragma unroll
        for (int h = 0; h < NH; ++h)
          if (w == 0 && run != 0xFFFFFFFFu && col_ok[h])
            storef4(a.huge_part + ((size_t)(base + run) * ngroups + g) * u.d + 64 * h + 4 * m, out[mb][h][v]);
      }
  }
  finish_table<16 * NH>(a, u, kind, k, base, nruns, ngroups);
}


int launch_segment_sort(const GroupArgs& g, hipStream_t st) {
  hipLaunchKernelGGL(segment_sort_kernel, dim3((unsigned)g.seg_tiles_max), dim3(kThreads), 0, st, g);
  DLRM_CHECK_LAUNCH();
  return DLRM_OK;
}

// Partial sums lie where nothing is left to read once the rows are grouped, if that holds more bag groups
// than the array laid out for them: the two arrays of the exported grouping or, for a weighted batch (whose
// records fill those), the partition's tile counts.
template <int G>
static int launch_hot(GroupArgs g, const UpdArgs& u, int kind, hipStream_t st) {
  constexpr int TB = kThreads / G * kHotStagePasses;    // bags of an LDS tile (weighted)
  constexpr int NH = G <= 16 ? 1 : G == 32 ? 2 : 4;
  const bool weighted = g.weights != nullptr;
  const int64_t room = weighted ? (int64_t)kMaxBuckets * g.nt_max * 4 : g.nnz * 8;   // bytes
  int64_t fit = room / (g.max_huge * u.d * 4);            // bag groups
  if (fit > hot_groups(g.B, u.d))
    g.huge_part = reinterpret_cast<float*>(weighted ? g.hist : g.seg_start);
  else
    fit = hot_groups(g.B, u.d);
  if (weighted) {
    // tiles per workgroup: enough workgroups for two per compute unit if every table has hot rows
    const int64_t tiles = ((int64_t)g.B + TB - 1) / TB;
    int64_t nt = (tiles * g.K + 511) / 512;
    if (nt > kHotTilesPerGroup) nt = kHotTilesPerGroup;
    while ((tiles + nt - 1) / nt > fit) ++nt;   // kHotTilesPerGroup tiles always fit
    const int ng = (int)((tiles + nt - 1) / nt);
    hipLaunchKernelGGL((hot_rows_weighted_kernel<G>), dim3(ng, g.K), dim3(kThreads), 0, st, g, u, kind, ng, (int)nt);
  } else {
    // bag groups at most: every table's share of the machine or groups of kHotGroupMin bags, within the room
    int64_t most = hot_slots(NH) / g.K;
    const int64_t small = ((int64_t)g.B + kHotGroupMin - 1) / kHotGroupMin, units = ((int64_t)g.B + kHotUnit - 1) / kHotUnit;
    if (most < small) most = small;
    if (most > hot_slots(NH)) most = hot_slots(NH);
    if (most > units) most = units;
    if (most > fit) most = fit;
    hipLaunchKernelGGL((hot_rows_dense_kernel<NH>), dim3((unsigned)most, g.K), dim3(kThreads), 0, st, g, u, kind);
  }
  DLRM_CHECK_LAUNCH();
  return DLRM_OK;
}

int launch_hot_rows(const GroupArgs& g, const UpdArgs& u, int G, int dtype, int opt, hipStream_t st) {
  const int kind = dtype * 2 + opt;
  switch (G) {
    case 1: return launch_hot<1>(g, u, kind, st);
    case 2: return launch_hot<2>(g, u, kind, st);
    case 4: return launch_hot<4>(g, u, kind, st);
    case 8: return launch_hot<8>(g, u, kind, st);
    case 16: return launch_hot<16>(g, u, kind, st);
    case 32: return launch_hot<32>(g, u, kind, st);
    case 64: return launch_hot<64>(g, u, kind, st);
  }
  return DLRM_ERR_BAD_SHAPE;
}

}  // namespace dlrm
