// Backward steps 4 / 4a and the row updates: sorted runs -> one read-modify-write per row.
// Template code; bwd_reduce_{sgd,adagrad}[_weighted].hip instantiate it per optimizer and per
// unweighted / weighted pooling.
#pragma once
#include "bwd_sort.h"

namespace dlrm {

// The second member of a sorted pair is the bag itself (sum pooling) or, for a weighted batch,
// the position inside the table, by which the bag and the weight a of Eq. (2) are looked up.
struct Entry {
  uint32_t bag;
  float w;
};
template <bool WT>
__device__ inline Entry entry_of(const GroupArgs& a, int64_t tbl, uint32_t val) {
  Entry e;
  if constexpr (WT) {
    const PosEntry pe = a.pos_entry[tbl + val];
    e.bag = pe.bag;
    e.w = pe.w;
  } else {
    e.bag = val;
    e.w = 1.0f;
  }
  return e;
}

// A weighted bucket sorted in LDS has its entries resolved once, by all threads at the same time,
// before any run is summed: the bag replaces the position in the sorted values and the weight goes to
// LDS beside it, in two pieces (the sort's per-wavefront counters, dead once the sort is done, and
// an extension for the rest), which keeps four workgroups per compute unit.  Without this every
// gradient row load waits for two dependent gathers of its own.
constexpr int kResolvedLo = kNW * kSortBuckets;
struct ResolvedW {
  float* lo;  // entries [0, kResolvedLo)
  float* hi;  // entries [kResolvedLo, kBktCap)
  __device__ float& at(uint32_t i) const { return i < (uint32_t)kResolvedLo ? lo[i] : hi[i - kResolvedLo]; }
};
// Runs longer than this are summed by the whole workgroup.  With many lane groups per workgroup
// (narrow rows) a medium run left to one lane group is the critical path of the bucket sooner.
template <int G>
__device__ constexpr uint32_t long_run() {
  return kThreads / G >= 32 ? (uint32_t)kLongRunMin : (uint32_t)kLongRun;
}

// Sum (weight times) dS rows of the sorted entries [i0, i1) taking every `stride`-th entry from
// i0 + first; U loads in flight, ascending order.  vals: LDS or global.  tbl: start of the table
// in the batch's index array.
template <int U, bool WT>
__device__ inline f32x4 sum_entries(const GroupArgs& a, int64_t tbl, const float* g, int64_t stride_b,
                                    const uint32_t* vals, uint32_t i0, uint32_t i1,
                                    uint32_t first, uint32_t stride) {
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  for (uint32_t i = i0 + first; i < i1; i += U * stride) {
    Entry e[U];
    f32x4 v[U];
#pragma unroll
    for (int t = 0; t < U; ++t) e[t] = entry_of<WT>(a, tbl, vals[i + t * stride < i1 ? i + t * stride : i]);
#pragma unroll
    for (int t = 0; t < U; ++t) v[t] = loadf4(g + (int64_t)e[t].bag * stride_b);
#pragma unroll
    for (int t = 0; t < U; ++t) {
      if (i + t * stride < i1) {
        if constexpr (WT) {
          acc.x = fmaf(e[t].w, v[t].x, acc.x);
          acc.y = fmaf(e[t].w, v[t].y, acc.y);
          acc.z = fmaf(e[t].w, v[t].z, acc.z);
          acc.w = fmaf(e[t].w, v[t].w, acc.w);
        } else {
          acc += v[t];
        }
      }
    }
  }
  return acc;
}

// keys/bags: the bucket's sorted pairs (n of them; LDS or global), heads: LDS list of run starts
// with heads[nruns] = n.  gpos0: global position of the bucket's first pair.
template <int DT, int G, int OPT, bool WT>
__device__ inline void reduce_runs(const GroupArgs& a, const UpdArgs& u, const Bucket& b, char* W,
                                   const uint32_t* keys, const uint32_t* bags, const uint32_t* heads,
                                   uint32_t h0, uint32_t nruns, const uint32_t* longs, uint32_t nlong,
                                   int src, float* part) {
  constexpr int NG = kThreads / G;
  // gradient rows a lane group keeps in flight while the workgroup sums a long run: few lane groups
  // (wide rows) need more each to keep the same number of bytes in flight
  constexpr int kLongU = (NG >= 32 || WT) ? 4 : 8;
  const int grp = threadIdx.x / G, chunk = threadIdx.x % G;
  const bool col_ok = chunk * 4 < u.d;
  // lanes past the last column shadow column group 0 (same addresses) and never write
  const float* g = u.dS + (int64_t)b.k * u.stride_k + (col_ok ? chunk : 0) * 4;
  // short runs: a lane group takes RU runs per round; the table rows and the first gradient
  // row of all RU runs are requested before any of them is consumed
  constexpr int RU = OPT == kAdagrad ? 2 : 4;  // Adagrad also holds the state rows
  const int cchunk = col_ok ? chunk : 0;
  float* const H = b.H;
  const int64_t tbl = WT ? a.tbl_off[b.k] : 0;
  for (uint32_t r0 = (uint32_t)grp * RU; r0 < nruns; r0 += NG * RU) {
    uint32_t i0[RU], i1[RU];
    RowRef wp[RU];
    RowVal wv[RU];
    f32x4 acc[RU];
#pragma unroll
    for (int t = 0; t < RU; ++t) {
      const uint32_t rr = r0 + t < nruns ? r0 + t : nruns - 1;  // the tail repeats the last run
      i0[t] = heads[rr] - h0;
      i1[t] = heads[rr + 1] - h0;
      wp[t] = row_ref<DT, OPT>(W, H, u.d, keys[i0[t]], cchunk);
    }
    Entry e0[RU];
#pragma unroll
    for (int t = 0; t < RU; ++t) e0[t] = entry_of<WT>(a, tbl, bags[i0[t]]);
#pragma unroll
    for (int t = 0; t < RU; ++t) acc[t] = loadf4(g + (int64_t)e0[t].bag * u.stride_b);
#pragma unroll
    for (int t = 0; t < RU; ++t) wv[t] = row_load<DT, OPT>(wp[t]);
    if constexpr (WT) {
#pragma unroll
      for (int t = 0; t < RU; ++t) acc[t] *= e0[t].w;
    }
#pragma unroll
    for (int t = 0; t < RU; ++t) {
      const uint32_t len = i1[t] - i0[t];
      if (r0 + t >= nruns || len > long_run<G>()) continue;
      if (len > 1) acc[t] += sum_entries<4, WT>(a, tbl, g, u.stride_b, bags, i0[t] + 1, i1[t], 0, 1);
      if (col_ok) row_update_store<DT, OPT>(wp[t], wv[t], acc[t], u);
    }
  }
  // long runs: the whole workgroup per run, lane group s taking entries s, s+NG, ...; the NG
  // partial sums are added in group order (in two levels of fixed shape when NG > 16)
  for (uint32_t q = 0; q < nlong; ++q) {  // uniform
    const uint32_t r = longs[q];
    const uint32_t i0 = heads[r] - h0, i1 = heads[r + 1] - h0;
    const uint32_t len = i1 - i0;
    if (len > (uint32_t)kHugeRun && a.no_tail && threadIdx.x == 0) atomicAdd(&b.route[kRouteHugeInPlace], 1u);
    if (len > (uint32_t)kHugeRun && !a.no_tail) {  // queue for the multi-workgroup pass
      if (threadIdx.x == 0) {
        HugeRun hr;
        hr.k = (uint32_t)b.k;
        hr.row = keys[i0];
        hr.start = b.start + h0 + i0;
        hr.len = len;
        hr.src = (uint32_t)src;
        hr.pad0 = hr.pad1 = hr.pad2 = 0;
        const uint32_t nth = atomicAdd(&a.hot_cnt[b.k], 1u);
        if (nth == 0u) atomicAdd(&a.seg_meta[kHotTables], 1u);
        a.huge_runs[hot_list_base(a, b.k) + nth] = hr;
      }
      continue;
    }
    // the row is requested first: its latency hides behind the gather
    const bool upd = grp == 0 && col_ok;
    RowRef wr = row_ref<DT, OPT>(W, H, u.d, keys[i0], cchunk);
    RowVal wv{};
    if (upd) wv = row_load<DT, OPT>(wr);
    const f32x4 acc = sum_entries<kLongU, WT>(a, tbl, g, u.stride_b, bags, i0, i1, (uint32_t)grp, (uint32_t)NG);
    __syncthreads();
    if (col_ok) storef4(part + grp * (G * 4) + chunk * 4, acc);
    __syncthreads();
    constexpr int L1 = NG > 16 ? 8 : 1;  // many lane groups: sums of L1 consecutive partials first
    if constexpr (L1 > 1) {
      if (grp < NG / L1 && col_ok) {
        f32x4 t = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < L1; ++s) t += loadf4(part + (grp * L1 + s) * (G * 4) + chunk * 4);
        storef4(part + grp * L1 * (G * 4) + chunk * 4, t);  // a slot only this lane reads above
      }
      __syncthreads();
    }
    if (upd) {
      f32x4 tot = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < NG / L1; ++s) tot += loadf4(part + s * L1 * (G * 4) + chunk * 4);
      row_update_store<DT, OPT>(wr, wv, tot, u);
    }
  }
}

// A bucket sorted in LDS, reduced with the WORK, not the runs, dealt evenly: lane
// group g takes the sorted entries [g*E, (g+1)*E), E = ceil(n / groups), whatever runs they belong
// to, U gradient rows in flight from the first entry to the last.  An entry whose row differs from
// its predecessor's starts a run (its table row is requested with the gradient rows of its round);
// a run that ends inside the slab is applied at once.  What a slab holds of a run that began in an
// earlier slab goes to LDS, and after one barrier the group where a run began adds the later slabs'
// pieces in slab order and applies the row.  Within a run the entries are added in position order
// inside each slab and the slabs in order: a fixed order, the same on every call.  No list of run
// heads is needed, and a run of any length inside the bucket is covered.
// WT: sval holds the resolved bags and rw the weights a of Eq. (2) of the sorted entries.
template <int DT, int G, int OPT, bool WT = false, bool KEEP = false>
__device__ inline void reduce_slabs(const UpdArgs& u, const Bucket& b, char* W, const uint32_t* skey,
                                    const uint32_t* sval, uint32_t n, float* part, uint32_t* flags,
                                    const ResolvedW& rw = ResolvedW{nullptr, nullptr}) {
  constexpr int NG = kThreads / G;
  // Gradient rows in flight per lane group, each measured with whole libraries on one box.  16-bit tables, SGD (128
  // registers): 3 / 4 / 6 / 8 / 10 -> 1.154 / 1.178 / 1.140 / 1.123 / 1.240 ms per launch on the hot-row workload.
  // fp32, SGD (168 registers): 4 / 8 / 12 -> 165 / 162 / 160 us on the multi-hot workload, step 135.8 / 134.3 /
  // 132.5 us on the large one-hot one (12 spills about 80 bytes, 16 three times that).  Adagrad: 6 and 8 are no different now that
  // a round's row requests do not wait for each other (state_base), and 6 needs fewer registers; before, 4 / 6 / 8 took
  // 2.66 / 2.40 / 2.57 ms on the hot-row workload.
  constexpr int U = OPT == kAdagrad ? 6 : DT == DLRM_F32 ? 12 : 8;
  const int grp = threadIdx.x / G, chunk = threadIdx.x % G;
  const bool col_ok = chunk * 4 < u.d;
  const int cchunk = col_ok ? chunk : 0;  // lanes past the last column shadow column group 0 and never write
  const float* g = u.dS + (int64_t)b.k * u.stride_k + cchunk * 4;
  float* const H = b.H;
  const uint32_t E = (n + NG - 1) / NG;
  const uint32_t p0 = (uint32_t)grp * E < n ? (uint32_t)grp * E : n;
  const uint32_t p1 = p0 + E < n ? p0 + E : n;
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 acc = zero, headp = zero;
  bool have = false;   // a run has begun in this slab
  RowRef cur{nullptr, nullptr};
  RowVal curv{};
  for (uint32_t c0 = p0; c0 < p1; c0 += U) {
    uint32_t key[U];
    bool hd[U];
    f32x4 v[U];
    float wt[WT ? U : 1];
    // the table rows of the runs that begin in this round (16-bit tables: 8 bytes per lane)
    u32x2 wlo[U], whi[DT == DLRM_F32 ? U : 1];
    f32x4 wh[OPT == kAdagrad ? U : 1];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const uint32_t p = c0 + j < p1 ? c0 + j : p1 - 1;
      key[j] = skey[p];
      const uint32_t prev = skey[p > 0 ? p - 1 : 0];
      hd[j] = c0 + j < p1 && (p == 0 || key[j] != prev);
      v[j] = loadf4(g + (int64_t)sval[p] * u.stride_b);
      if constexpr (WT) wt[j] = rw.at(p);
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      wlo[j] = u32x2{0u, 0u};
      if constexpr (DT == DLRM_F32) whi[j] = u32x2{0u, 0u};
      if constexpr (OPT == kAdagrad) wh[j] = zero;
      if (hd[j]) {
        const RowVal t = row_load<DT, OPT, KEEP>(row_ref<DT, OPT>(W, H, u.d, key[j], cchunk));
        wlo[j] = u32x2{t.w.x, t.w.y};
        if constexpr (DT == DLRM_F32) whi[j] = u32x2{t.w.z, t.w.w};
        if constexpr (OPT == kAdagrad) wh[j] = t.h;
      }
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (hd[j]) {
        if (have) {
          if (col_ok) row_update_store<DT, OPT>(cur, curv, acc, u);
        } else {
          headp = acc;
        }
        acc = zero;
        cur = row_ref<DT, OPT>(W, H, u.d, key[j], cchunk);
        curv.w = u32x4{wlo[j].x, wlo[j].y, 0u, 0u};
        if constexpr (DT == DLRM_F32) {
          curv.w.z = whi[j].x;
          curv.w.w = whi[j].y;
        }
        if constexpr (OPT == kAdagrad) curv.h = wh[j];
        have = true;
      }
      if (c0 + j < p1) {
        if constexpr (WT) {
          acc.x = fmaf(wt[j], v[j].x, acc.x);
          acc.y = fmaf(wt[j], v[j].y, acc.y);
          acc.z = fmaf(wt[j], v[j].z, acc.z);
          acc.w = fmaf(wt[j], v[j].w, acc.w);
        } else {
          acc += v[j];
        }
      }
    }
  }
  if (!have) headp = acc;   // the whole slab continues an earlier run (an empty slab: zero)
  if (col_ok) storef4(part + grp * (G * 4) + chunk * 4, headp);
  if (chunk == 0) flags[grp] = p0 < p1 ? (have ? 1u : 2u) : 0u;   // empty / a run begins here / all continuation
  __syncthreads();
  if (have) {
    f32x4 tot = acc;
    if constexpr (NG < 32) {
      for (int g2 = grp + 1; g2 < NG; ++g2) {
        const uint32_t f = flags[g2];
        if (f == 0u) break;
        tot += loadf4(part + g2 * (G * 4) + cchunk * 4);
        if (f == 1u) break;
      }
    } else {
      // With narrow rows a long run spans up to 255 slabs.  The two next ones, which most runs end in, are read at once, those
      // behind them kAhead at a time, not each once the one before has said that the run goes on.  Update alone, 26 tables
      // of 8192 skewed lookups, one by one / now: fp32 d = 4 101 / 71 us, d = 8 73.4 / 61.1, fp16 d = 8 72.8 / 59.5; of 2048:
      // 36.2 / 23.2, 24.0 / 16.7, 22.3 / 16.4; 27 fp32 tables of 2900 uniform lookups, d = 4: one, then eight 32.0, two, then
      // eight 31.5.  Rows of 64 columns and more (up to 15 slabs) have nothing to gain, and the registers for it are spilled:
      // pooling + update, one table, 24 bags of 73 on 8 rows, d = 156, as above / so 39.5 / 40.8.
      constexpr int kAhead = 8;
      const int g1 = grp + 1 < NG ? grp + 1 : NG - 1, gn = grp + 2 < NG ? grp + 2 : NG - 1;
      uint32_t f = flags[g1], fn = flags[gn];
      const f32x4 next = loadf4(part + g1 * (G * 4) + cchunk * 4), after = loadf4(part + gn * (G * 4) + cchunk * 4);
      f = grp + 1 < NG ? f : 0u;
      fn = grp + 2 < NG ? fn : 0u;
      if (f != 0u) tot += next;
      f = f == 2u ? fn : 0u;
      if (f != 0u) tot += after;
      for (int g2 = grp + 3; f == 2u; g2 += kAhead) {
        uint32_t fs[kAhead];
        f32x4 more[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
          const int gj = g2 + j < NG ? g2 + j : NG - 1;
          fs[j] = g2 + j < NG ? flags[gj] : 0u;
          more[j] = loadf4(part + gj * (G * 4) + cchunk * 4);
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {   // branch-free: behind the run's end f is 0 or 1, and the identity is added
          f = f == 2u ? fs[j] : 0u;
          const bool in = f != 0u;
          tot += f32x4{in ? more[j].x : -0.0f, in ? more[j].y : -0.0f, in ? more[j].z : -0.0f, in ? more[j].w : -0.0f};
        }
      }
    }
    if (col_ok) row_update_store<DT, OPT>(cur, curv, tot, u);
  }
}

// Weighted: every sorted entry is resolved (position -> bag, weight) once, by all threads at the same time.  All of a thread's
// entries are requested together: none behind a branch, since each of those waits for the loads before it, up to eight round
// trips a bucket.  A slot past the end reads the table's first entry and is written like the others; nothing reads it.
__device__ inline void resolve_sorted(const GroupArgs& a, int k, uint32_t* sval, uint32_t n, const ResolvedW& rw) {
  const PosEntry* const pe = a.pos_entry + a.tbl_off[k];
  PosEntry e[kBktItems];
#pragma unroll
  for (int j = 0; j < kBktItems; ++j) {
    const uint32_t li = threadIdx.x + j * kThreads, pos = sval[li];
    e[j] = pe[li < n ? pos : 0u];
  }
#pragma unroll
  for (int j = 0; j < kBktItems; ++j) {  // a thread rewrites only the slots it read
    const uint32_t li = threadIdx.x + j * kThreads;
    sval[li] = e[j].bag;
    rw.at(li) = e[j].w;
  }
  __syncthreads();
}

// Run heads of sorted keys[0..n) (LDS) into s.heads (positions, ascending) with the sentinel
// heads[nruns] = n.  Returns nruns.  All threads call it.
__device__ inline uint32_t compact_heads_lds(SortLds& s, int n) {
  const int tid = threadIdx.x;
  uint32_t flags = 0, cnt = 0;
#pragma unroll
  for (int j = 0; j < kBktItems; ++j) {
    const int li = tid * kBktItems + j;
    if (li < n && (li == 0 || s.skey[li] != s.skey[li - 1])) {
      flags |= 1u << j;
      ++cnt;
    }
  }
  uint32_t total;
  uint32_t pos = block_exclusive_scan<kThreads>(cnt, s.smem, &total);
#pragma unroll
  for (int j = 0; j < kBktItems; ++j) {
    if (flags & (1u << j)) s.heads[pos++] = (uint32_t)(tid * kBktItems + j);
  }
  if (tid == 0) s.heads[total] = (uint32_t)n;
  __syncthreads();
  return total;
}

// Lists the runs longer than `longer_than` (>= kLongRunMin) among s.heads[0..nruns] (any order: each is a
// different row).  At most kBktCap/kLongRunMin + 1 of them have their head inside a window of kBktCap
// positions.
__device__ inline uint32_t collect_long_runs(SortLds& s, uint32_t nruns, uint32_t longer_than) {
  if (threadIdx.x == 0) s.nlong = 0;
  __syncthreads();
  for (uint32_t r = threadIdx.x; r < nruns; r += kThreads) {
    if (s.heads[r + 1] - s.heads[r] > longer_than) s.longs[atomicAdd(&s.nlong, 1u)] = r;
  }
  __syncthreads();
  return s.nlong;
}

// First position in [lo, n) whose key differs from `key`, given that keys are sorted and every
// position in [.., lo) of the run equals it: 256-ary search, workgroup-uniform.
__device__ inline uint32_t run_end_search(const uint32_t* keys, uint32_t lo, uint32_t n, uint32_t key) {
  uint32_t hi = n;  // the answer lies in [lo, hi]
  while (lo < hi) {
    const uint32_t step = (hi - lo + kThreads - 1) / kThreads;
    const uint32_t q = lo + threadIdx.x * step;
    const int same = (q < hi && keys[q] == key) ? 1 : 0;
    const uint32_t cnt = (uint32_t)__syncthreads_count(same);  // sorted: the first cnt probes match
    if (cnt == 0) break;
    const uint32_t nhi = lo + cnt * step < hi ? lo + cnt * step : hi;
    lo = lo + (cnt - 1) * step + 1;
    hi = nhi;
  }
  return lo;
}

// One window of kBktCap positions of a sorted pair list (global memory): the runs whose head
// lies in the window are reduced and applied; a run may extend past the window.
template <int DT, int G, int OPT, bool WT>
__device__ inline void reduce_window(const GroupArgs& a, const UpdArgs& u, const Bucket& b, char* W,
                                     const uint32_t* keys, const uint32_t* bags, uint32_t w0, int src,
                                     SortLds& s, float* part) {
  const int cnt = (int)(b.n - w0 < (uint32_t)kBktCap ? b.n - w0 : (uint32_t)kBktCap);
  const int tid = threadIdx.x;
  uint32_t flags = 0, c = 0;
#pragma unroll
  for (int j = 0; j < kBktItems; ++j) {
    const int li = tid * kBktItems + j;
    if (li < cnt && (w0 + li == 0 || keys[w0 + li] != keys[w0 + li - 1])) {
      flags |= 1u << j;
      ++c;
    }
  }
  uint32_t total;
  uint32_t pos = block_exclusive_scan<kThreads>(c, s.smem, &total);
#pragma unroll
  for (int j = 0; j < kBktItems; ++j) {
    if (flags & (1u << j)) s.heads[pos++] = w0 + (uint32_t)(tid * kBktItems + j);
  }
  __syncthreads();
  if (total > 0) {  // uniform
    const uint32_t e = run_end_search(keys, w0 + (uint32_t)cnt, b.n, keys[s.heads[total - 1]]);
    if (tid == 0) s.heads[total] = e;
    __syncthreads();
    const uint32_t nlong = collect_long_runs(s, total, long_run<G>());
    reduce_runs<DT, G, OPT, WT>(a, u, b, W, keys, bags, s.heads, 0u, total, s.longs, nlong, src, part);
  }
  __syncthreads();
}

// A value that is the same in all lanes, though the compiler cannot see it (it came out of LDS, or from threadIdx): loops and addresses that
// depend on it are scalar.
__device__ inline uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// --- 4a. oversized buckets: dominant rows split off first ------------------------------------------
// A bucket outgrows the LDS sort almost always because a few hot rows own most of its pairs.
// Rows holding at least kCandMin of the bucket's first kBktCap pairs become candidates (at most
// kCand = kBktCap / kCandMin of them).  One count pass and one stable partition pass over the
// bucket then give every candidate its own list (position order is kept, so its bags ascend) and
// collect the rest behind them; no pair of a candidate is ever sorted.  The rest usually fits
// the LDS sort; if not, it alone goes to the segment kernels or the streaming sort.
struct SplitLds {
  uint32_t cand[kCand];       // candidate row ids, in row order; unused slots 0xFFFFFFFF
  uint32_t cnt[kCand + 1];    // pairs per class; class kCand = every other row
  uint32_t wcnt[kNW][kCand + 1];   // the same per wavefront (each streams a quarter of the bucket)
  uint32_t wbase[kNW][kCand + 1];  // first destination of every (wavefront, class)
  uint32_t cbase[kCand + 2];  // exclusive prefix of cnt
  uint32_t nc;
};

// Pairs [bk.start, bk.start + bk.n) of pair buffer src, more than kBktCap of them, that no
// shortcut applies to: queued as a segment when per-row counters fit LDS, else sorted here.
template <int DT, int G, int OPT, bool WT>
__device__ inline void sort_reduce_large(const GroupArgs& a, const UpdArgs& u, const Bucket& bk, char* W,
                                         int src, SortLds& s, float* part) {
  if (bk.low_bits <= kSegMaxBits && !a.no_tail) {
    if (threadIdx.x == 0) {
      const uint32_t nt = (bk.n + kBktCap - 1) / kBktCap;
      // one 64-bit counter hands out the slot and the first tile together, so that the list is
      // ordered by first tile
      const unsigned long long old =
          atomicAdd(reinterpret_cast<unsigned long long*>(a.seg_meta), (1ull << 32) | (unsigned long long)nt);
      SegInfo sg;
      sg.start = bk.start;
      sg.n = bk.n;
      sg.k = (uint32_t)bk.k;
      sg.low_bits = (uint32_t)bk.low_bits;
      sg.tile0 = (uint32_t)old;
      sg.src = (uint32_t)src;
      sg.pad1 = sg.pad2 = 0;
      a.segs[(uint32_t)(old >> 32)] = sg;
    }
    return;
  }
  if (threadIdx.x == 0) atomicAdd(&bk.route[kRouteGlobalSort], 1u);
  const int res = sort_bucket_global(a, bk, s, src);
  __syncthreads();
  const uint32_t* keys = a.keys[res] + bk.start;
  const uint32_t* bags = a.vals[res] + bk.start;
  for (uint32_t w0 = 0; w0 < bk.n; w0 += kBktCap) reduce_window<DT, G, OPT, WT>(a, u, bk, W, keys, bags, w0, res, s, part);
}

template <int DT, int G, int OPT, bool WT>
__device__ inline void reduce_oversized(const GroupArgs& a, const UpdArgs& u, const Bucket& b, char* W,
                                        SortLds& s, SplitLds& sp, float* part, const ResolvedW& rw) {
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  // ---- candidates: long runs among the first kBktCap pairs
  if (tid < kCand) sp.cand[tid] = 0xFFFFFFFFu;
  {
    Bucket head = b;
    head.n = (uint32_t)kBktCap;
    sort_bucket_lds(a, head, s, 1);
    const uint32_t nruns = compact_heads_lds(s, kBktCap);
    uint32_t flags = 0, c = 0;
#pragma unroll
    for (int j = 0; j < kBktItems; ++j) {  // thread t owns runs [t*kBktItems, (t+1)*kBktItems): row order
      const uint32_t r = (uint32_t)(tid * kBktItems + j);
      if (r < nruns && s.heads[r + 1] - s.heads[r] >= (uint32_t)kCandMin) {
        flags |= 1u << j;
        ++c;
      }
    }
    uint32_t total;
    uint32_t pos = block_exclusive_scan<kThreads>(c, s.smem, &total);
#pragma unroll
    for (int j = 0; j < kBktItems; ++j)
      if (flags & (1u << j)) sp.cand[pos++] = s.skey[s.heads[tid * kBktItems + j]];
    if (tid == 0) sp.nc = total;
  }
  __syncthreads();
  const uint32_t nc = sp.nc;
  if (nc == 0) {  // uniform
    sort_reduce_large<DT, G, OPT, WT>(a, u, b, W, 1, s, part);
    return;
  }
  if (tid == 0) atomicAdd(&b.route[kRouteSplit], 1u);
  uint32_t cd[kCand];   // scalars, as are the counts below
#pragma unroll
  for (int c = 0; c < kCand; ++c) cd[c] = uniform(sp.cand[c]);
  const uint32_t* kin = a.keys[1] + b.start;
  const uint32_t* vin = a.vals[1] + b.start;
  constexpr uint32_t kNone = 0xFFFFFFFFu;   // no row
  // Both passes: wavefront w streams its own quarter [q0, q1) of the bucket, no barriers inside, 8 steps of 64 pairs
  // at a time, the next 8 in flight.  A candidate costs a comparison of a step and the count of the lanes that agree.
  const uint32_t span = (b.n + kNW * DLRM_WAVE - 1) / (kNW * DLRM_WAVE) * DLRM_WAVE;
  const uint32_t q0 = uniform((uint32_t)w * span < b.n ? (uint32_t)w * span : b.n);
  const uint32_t q1 = uniform(q0 + span < b.n ? q0 + span : b.n);
  // ---- pass 1: pairs per (wavefront, class)
  uint32_t cn[kCand], key[8];
#pragma unroll
  for (int c = 0; c < kCand; ++c) cn[c] = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const uint32_t i = q0 + q * DLRM_WAVE + lane;
    key[q] = kin[i < q1 ? i : q1 - 1u];
    key[q] = i < q1 ? key[q] : kNone;
  }
  for (uint32_t i0 = q0; i0 < q1; i0 += DLRM_WAVE * 8) {
    uint32_t nk[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t i = i0 + DLRM_WAVE * 8 + q * DLRM_WAVE + lane;
      nk[q] = kin[i < q1 ? i : q1 - 1u];
      nk[q] = i < q1 ? nk[q] : kNone;
    }
#pragma unroll
    for (int c = 0; c < kCand; ++c) {
      if ((uint32_t)c < nc) {  // uniform
#pragma unroll
        for (int q = 0; q < 8; ++q) cn[c] += (uint32_t)__popcll(__ballot(key[q] == cd[c]));
      }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) key[q] = nk[q];
  }
  if (lane == 0) {
    uint32_t rest = q1 - q0;
#pragma unroll
    for (int c = 0; c < kCand; ++c) {
      sp.wcnt[w][c] = cn[c];
      rest -= cn[c];
    }
    sp.wcnt[w][kCand] = rest;
  }
  __syncthreads();
  if (tid <= kCand) {
    uint32_t tot = 0;
    for (int i = 0; i < kNW; ++i) tot += sp.wcnt[i][tid];
    sp.cnt[tid] = tot;
  }
  __syncthreads();
  if (tid == 0) {
    uint32_t run = 0;
    for (int c = 0; c <= kCand; ++c) {
      sp.cbase[c] = run;
      run += sp.cnt[c];
    }
    sp.cbase[kCand + 1] = run;
  }
  __syncthreads();
  if (tid <= kCand) {  // where wavefront i's first pair of the class goes
    uint32_t run = sp.cbase[tid];
    for (int i = 0; i < kNW; ++i) {
      sp.wbase[i][tid] = run;
      run += sp.wcnt[i][tid];
    }
  }
  __syncthreads();
  // ---- pass 2: stable partition by class into pair buffer 0.  Candidate lists keep only the
  // bags (plus the row id at their first position); the rest keeps (row, bag).  Within a step
  // of 64 pairs the lanes of one class rank themselves by ballot; the wavefront's running
  // destination per class is a scalar.
  uint32_t* kout = a.keys[0] + b.start;
  uint32_t* vout = a.vals[0] + b.start;
  uint32_t val[8], rest = uniform(sp.wbase[w][kCand]);
#pragma unroll
  for (int c = 0; c < kCand; ++c) cn[c] = uniform(sp.wbase[w][c]);   // the wavefront's running destinations
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const uint32_t i = q0 + q * DLRM_WAVE + lane;
    key[q] = kin[i < q1 ? i : q1 - 1u];
    key[q] = i < q1 ? key[q] : kNone;
    val[q] = vin[i < q1 ? i : q1 - 1u];
  }
  for (uint32_t i0 = q0; i0 < q1; i0 += DLRM_WAVE * 8) {
    uint32_t nk[8], nv[8], dst[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t i = i0 + DLRM_WAVE * 8 + q * DLRM_WAVE + lane;
      nk[q] = kin[i < q1 ? i : q1 - 1u];
      nk[q] = i < q1 ? nk[q] : kNone;
      nv[q] = vin[i < q1 ? i : q1 - 1u];
      dst[q] = kNone;
    }
#pragma unroll
    for (int c = 0; c < kCand; ++c) {
      if ((uint32_t)c < nc) {  // uniform
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const bool mine = key[q] == cd[c];
          const unsigned long long m = __ballot(mine);
          const uint32_t at = cn[c] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
          dst[q] = mine ? at : dst[q];
          cn[c] += (uint32_t)__popcll(m);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const bool other = key[q] != kNone && dst[q] == kNone;
      const unsigned long long m = __ballot(other);
      if (other) {
        dst[q] = rest + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        kout[dst[q]] = key[q];
      }
      rest += (uint32_t)__popcll(m);
      if (key[q] != kNone) vout[dst[q]] = val[q];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      key[q] = nk[q];
      val[q] = nv[q];
    }
  }
  __syncthreads();
  if ((uint32_t)tid < nc) kout[sp.cbase[tid]] = sp.cand[tid];
  if ((uint32_t)tid <= nc) s.heads[tid] = sp.cbase[tid];
  __syncthreads();
  // ---- candidate lists are runs: those above kHugeRun are queued as hot rows, the others reduced like sorted buckets, as
  // many whole runs at a time as LDS holds.  Bound by the round trips of one workgroup on which the launch waits.  With run
  // after run (two barriers and a chain of list and row loads each), classes found by a loop over those present in a step and
  // their destinations in LDS / now: 26 bf16 tables of 41 K skewed lookups 90 / 81 us for the kernel, 100 fp16 tables with
  // Adagrad 60 / 50 us (with the state's base as a scalar).  The entries of a group of runs are requested together, and one
  // pass over the runs' starts gives all of them their rows; each entry's read and search by itself, update alone, 26 fp32
  // tables of 8192 skewed lookups: d = 4 74.1 / 71.1 us, d = 12 60.1 / 56.9, d = 64 66.2 / 64.2.
  // Rows are read streaming here, also where they share sectors (KEEP).  Streaming / plain loads, 27 updates of such tables: from
  // 1 % in favour of plain ones to 3 % against (26 x 41 K skewed lookups, us: fp32 d = 36 181.9 / 180.8, weighted 255.1 / 256.9,
  // fp16 Adagrad d = 40 230.2 / 235.5).
  {
    const uint32_t nlong = collect_long_runs(s, nc, (uint32_t)kHugeRun);
    if (nlong != 0)
      reduce_runs<DT, G, OPT, WT>(a, u, b, W, kout, vout, s.heads, 0u, 0u, s.longs, nlong, 0, part);
  }
  // (a run between the two limits would be queued and reduced here as well, one beyond the larger limit neither)
  static_assert(kHugeRun == kBktCap, "a run is queued or fits LDS, never both");
  for (uint32_t c0 = 0; c0 <= nc;) {   // uniform; last, as class nc, the rest
    uint32_t c1 = c0, n = 0;
    if (c0 < nc) {
      while (c1 < nc && n + uniform(sp.cnt[c1]) <= (uint32_t)kBktCap) n += uniform(sp.cnt[c1++]);
      if (n == 0) {   // a queued run
        ++c0;
        continue;
      }
      const uint32_t from = uniform(sp.cbase[c0]);
      uint32_t t0 = threadIdx.x;
      asm("" : "+v"(t0));   // entry addresses are made here: hoisted to the kernel's start they would be spilled until now
      uint32_t row[kBktItems], bag[kBktItems];   // (weighted: positions)
#pragma unroll
      for (int j = 0; j < kBktItems; ++j) {   // requested together; a slot past the end re-reads the last entry
        const uint32_t li = t0 + j * kThreads;
        bag[j] = vout[from + (li < n ? li : n - 1u)];
        row[j] = 0u;
      }
      for (uint32_t c = c0; c < c1; ++c) {
        const uint32_t first = uniform(sp.cbase[c]) - from, id = uniform(sp.cand[c]);
#pragma unroll
        for (int j = 0; j < kBktItems; ++j) row[j] = (uint32_t)(t0 + j * kThreads) >= first ? id : row[j];
      }
      __syncthreads();   // the previous entries have been read
#pragma unroll
      for (int j = 0; j < kBktItems; ++j) {
        s.skey[t0 + j * kThreads] = row[j];
        s.sval[t0 + j * kThreads] = bag[j];
      }
    } else {
      Bucket others = b;
      others.start = b.start + uniform(sp.cbase[kCand]);
      others.n = n = uniform(sp.cnt[kCand]);
      if (n == 0) return;
      __syncthreads();
      if (n > (uint32_t)kBktCap) {
        sort_reduce_large<DT, G, OPT, WT>(a, u, others, W, 0, s, part);
        return;
      }
      sort_bucket_lds(a, others, s, 0);
      c1 = nc + 1;
    }
    __syncthreads();
    if constexpr (WT) resolve_sorted(a, b.k, s.sval, n, rw);
    reduce_slabs<DT, G, OPT, WT>(u, b, W, s.skey, s.sval, n, part, s.heads, rw);
    c0 = c1;
  }
}

// A bucket of more than kBktCap pairs (pair buffer 1).
template <int DT, int G, int OPT, bool WT>
__device__ inline void reduce_beyond_lds(const GroupArgs& a, const UpdArgs& u, const Bucket& b, char* W, SortLds& s,
                                         SplitLds& sp, float* part, const ResolvedW& rw) {
  if (b.low_bits == 0) {  // the bucket holds one row: a single run, already in position order
    if (threadIdx.x == 0) {
      s.heads[0] = 0;
      s.heads[1] = b.n;
      atomicAdd(&b.route[kRouteOneRow], 1u);
    }
    __syncthreads();
    const uint32_t nlong = collect_long_runs(s, 1, long_run<G>());
    reduce_runs<DT, G, OPT, WT>(a, u, b, W, a.keys[1] + b.start, a.vals[1] + b.start, s.heads, 0u, 1, s.longs, nlong, 1,
                       part);
    return;
  }
  reduce_oversized<DT, G, OPT, WT>(a, u, b, W, s, sp, part, rw);
}

template <int DT, int G, int OPT, bool WT, bool KEEP>
// register budget: 4 wavefronts per SIMD for 16-bit tables with SGD, 3 (168 registers) otherwise -- measured both ways
// on the multi-hot and one-hot workloads (fp32: 3 is 2 % ahead) and on the hot-row one (fp16: 4 is 12 % ahead)
__global__ __launch_bounds__(kThreads, (OPT == kAdagrad || DT == DLRM_F32) ? 3 : 4) void bucket_reduce_kernel(GroupArgs a, UpdArgs u) {
  __shared__ SortLds s;
  __shared__ SplitLds sp;
  __shared__ float part[kThreads * 4];
  __shared__ float wext[WT ? kBktCap - kResolvedLo : 1];
  uint32_t bid;
  bool listed;
  if (!bucket_id_of_block(a, &bid, &listed)) return;
  Bucket b = bucket_of_block(a, bid);
  if (b.n == 0 || (!listed && b.n > a.big)) return;   // a heavy bucket belongs to one of the first workgroups
  char* W = static_cast<char*>(u.tables[b.k]);
  b.H = state_base<OPT>(u, b.k);
  const ResolvedW rw{reinterpret_cast<float*>(&s.wcnt[0][0]), wext};
  if (b.n <= (uint32_t)kBktCap) {
    sort_bucket_lds(a, b, s);
    if constexpr (WT) resolve_sorted(a, b.k, s.sval, b.n, rw);
    reduce_slabs<DT, G, OPT, WT, KEEP>(u, b, W, s.skey, s.sval, b.n, part, s.heads, rw);
    return;
  }
  reduce_beyond_lds<DT, G, OPT, WT>(a, u, b, W, s, sp, part, rw);
}

// --- 4, small batches: no partition --------------------------------------------------------------
// Bag of a position of table k: binary search in kThreads evenly spaced offsets held in LDS, then
// between two of them in memory (bags may be empty: the last bag that starts at or before the position).
struct BagSearch {
  const int64_t* off;   // offsets of the table, B + 1 of them
  const uint32_t* smp;  // LDS: off[i * step], i < nsmp
  uint32_t B, nsmp, step, fixed;   // fixed: lookups per bag if the count divides evenly, else 0
  // N positions at once, so that their probes are in flight together; bags of one length need one guess each instead
  // of a chain of probes
  template <int N>
  __device__ void find_all(const uint32_t* pos, uint32_t* bag) const {
    if (step > 2 && fixed != 0) {   // uniform
      uint32_t lo[N], hi[N];
      bool good = true;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        bag[j] = fixed == 1 ? pos[j] : pos[j] / fixed;
        lo[j] = (uint32_t)off[bag[j]];
        hi[j] = (uint32_t)off[bag[j] + 1];
      }
#pragma unroll
      for (int j = 0; j < N; ++j) good = good && lo[j] <= pos[j] && pos[j] < hi[j];
      if (__all(good)) return;
    }
    uint32_t c[N];
#pragma unroll
    for (int j = 0; j < N; ++j) c[j] = 0;
#pragma unroll
    for (uint32_t w = kThreads / 2; w > 0; w >>= 1) {
      uint32_t v[N];
#pragma unroll
      for (int j = 0; j < N; ++j) v[j] = smp[c[j] + w < nsmp ? c[j] + w : nsmp - 1];
#pragma unroll
      for (int j = 0; j < N; ++j) c[j] += c[j] + w < nsmp && v[j] <= pos[j] ? w : 0u;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) bag[j] = c[j] * step;
    for (uint32_t w = step >> 1; w > 0; w >>= 1) {
      uint32_t v[N];
#pragma unroll
      for (int j = 0; j < N; ++j) v[j] = (uint32_t)off[bag[j] + w < B ? bag[j] + w : B];
#pragma unroll
      for (int j = 0; j < N; ++j)
        bag[j] += bag[j] + w < B && v[j] <= pos[j] ? w : 0u;
    }
  }
};

// Lookups [0, nk) of a table, nk <= kBktCap, whose row has the partition digit dg: rows and positions to s.skey / s.sval in
// position order.  Wavefront w takes positions [w * 512, w * 512 + 512).  Returns their number.  All threads call it.
template <typename IT>
__device__ inline uint32_t pick_lookups(const IT* idx, uint32_t nk, uint32_t dg, int shift, SortLds& s) {
  const int lane = lane_id(), w = wave_id();
  const unsigned long long lt = (1ull << lane) - 1ull;
  const uint32_t first = (uint32_t)(w * (DLRM_WAVE * kBktItems) + lane);
  uint32_t key[kBktItems], rank[kBktItems], mine = 0, before = 0, all = 0;
  bool hit[kBktItems];
#pragma unroll
  for (int j = 0; j < kBktItems; ++j) {
    const uint32_t p = first + j * DLRM_WAVE;
    key[j] = (uint32_t)idx[p < nk ? p : nk - 1];
  }
#pragma unroll
  for (int j = 0; j < kBktItems; ++j) {
    hit[j] = first + j * DLRM_WAVE < nk && key[j] >> shift == dg;
    const unsigned long long m = __ballot(hit[j]);
    rank[j] = mine + (uint32_t)__popcll(m & lt);
    mine += (uint32_t)__popcll(m);
  }
  if (lane == 0) s.longs[w] = mine;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kNW; ++i) {
    const uint32_t c = s.longs[i];
    before += i < w ? c : 0u;
    all += c;
  }
#pragma unroll
  for (int j = 0; j < kBktItems; ++j) {
    if (!hit[j]) continue;
    s.skey[before + rank[j]] = key[j];
    s.sval[before + rank[j]] = first + j * DLRM_WAVE;
  }
  return all;
}

// The same for any number of lookups up to kSmallBatch, in two steps: mark_lookups sets a bit per lookup in s.skey, without
// barriers and with kMarkItems loads of a lane in flight; marked_positions turns the bits into positions.  Bound by the
// issue of one wavefront per SIMD: 1 us per 4096 lookups (twice the loads in flight: slower).  Passing the row ids 2048 at
// a time instead, with a barrier each, and twice where the bucket outgrows the LDS sort, took 46 / 66 / 206 us where this
// takes 38 / 57 / 155 us (updates of 8, 16, 16 tables with 28000, 45000, 60000 lookups in one of them, d = 64).
constexpr int kMarkItems = 16;
static_assert(kSmallBatch <= kBktCap * 32 && kSmallBatch % (DLRM_WAVE * kMarkItems) == 0, "a bit per lookup in SortLds::skey");

// One wavefront's share of a round, kMarkItems words from word c0 on; FULL: none of its lookups lies beyond nk.  Bits beyond
// nk stay clear.  Returns how many rows have a smaller digit.
template <bool FULL, typename IT>
__device__ inline uint32_t mark_words(const IT* idx, uint32_t nk, uint32_t c0, uint32_t dg, int shift,
                                      unsigned long long* mask) {
  const uint32_t lane = (uint32_t)lane_id(), left = nk - c0 * DLRM_WAVE;
  const IT* from = idx + c0 * DLRM_WAVE;
  uint32_t key[kMarkItems], below = 0, lo = 0, hi = 0;
#pragma unroll
  for (int j = 0; j < kMarkItems; ++j) {
    const uint32_t p = j * DLRM_WAVE + lane;
    key[j] = (uint32_t)from[FULL || p < left ? p : left - 1];
  }
#pragma unroll
  for (int j = 0; j < kMarkItems; ++j) {
    const bool valid = FULL || j * DLRM_WAVE + lane < left;
    const uint32_t kd = key[j] >> shift;
    const unsigned long long m = __ballot(valid && kd == dg);
    below += (uint32_t)__popcll(__ballot(valid && kd < dg));
    lo = lane == (uint32_t)j ? (uint32_t)m : lo;
    hi = lane == (uint32_t)j ? (uint32_t)(m >> 32) : hi;
  }
  if (lane < (uint32_t)kMarkItems) mask[c0 + lane] = ((unsigned long long)hi << 32) | lo;
  return below;
}

// Returns how many rows with a smaller digit this wavefront saw.
template <typename IT>
__device__ inline uint32_t mark_lookups(const IT* idx, uint32_t nk, uint32_t dg, int shift, unsigned long long* mask) {
  uint32_t below = 0;
  for (uint32_t c0 = uniform(wave_id()) * kMarkItems; c0 * DLRM_WAVE < nk; c0 += kNW * kMarkItems) {
    below += (c0 + kMarkItems) * DLRM_WAVE <= nk ? mark_words<true>(idx, nk, c0, dg, shift, mask)
                                                 : mark_words<false>(idx, nk, c0, dg, shift, mask);
  }
  return below;
}

// A thread takes consecutive words of the mask: their set bits, and put(before + i, position) for the i-th of them.
__device__ inline uint32_t marked_words(uint32_t nk) { return ((nk + DLRM_WAVE - 1) / DLRM_WAVE + kThreads - 1) / kThreads; }
__device__ inline uint32_t count_marked(const unsigned long long* mask, uint32_t nk) {
  const uint32_t words = (nk + DLRM_WAVE - 1) / DLRM_WAVE, per = marked_words(nk);
  uint32_t n = 0;
  for (uint32_t q = threadIdx.x * per; q < (threadIdx.x + 1) * per && q < words; ++q) n += (uint32_t)__popcll(mask[q]);
  return n;
}
template <typename PUT>
__device__ inline void marked_positions(const unsigned long long* mask, uint32_t nk, uint32_t before, PUT put) {
  const uint32_t words = (nk + DLRM_WAVE - 1) / DLRM_WAVE, per = marked_words(nk);
  for (uint32_t q = threadIdx.x * per; q < (threadIdx.x + 1) * per && q < words; ++q) {
    for (unsigned long long m = mask[q]; m != 0ull; m &= m - 1ull)
      put(before++, q * DLRM_WAVE + (uint32_t)__ffsll((long long)m) - 1u);
  }
}

// rows[i] = idx[pos[i]], i < n
template <typename IT>
__device__ inline void rows_of_positions(const IT* idx, const uint32_t* pos, uint32_t n, uint32_t* rows) {
  for (uint32_t i0 = 0; i0 < n; i0 += kBktCap) {
    uint32_t p[kBktItems], row[kBktItems];
#pragma unroll
    for (int j = 0; j < kBktItems; ++j) {
      const uint32_t i = i0 + threadIdx.x + j * kThreads;
      p[j] = pos[i < n ? i : n - 1];
    }
#pragma unroll
    for (int j = 0; j < kBktItems; ++j) row[j] = (uint32_t)idx[p[j]];
#pragma unroll
    for (int j = 0; j < kBktItems; ++j) {
      const uint32_t i = i0 + threadIdx.x + j * kThreads;
      if (i < n) rows[i] = row[j];
    }
  }
}

// A batch of few lookups (GroupArgs::direct) has no steps 1-3: the workgroup of bucket (table, digit) reads all row ids
// of the table and keeps its own.  The row ids are read once per bucket, from L2 (a few MB in all), in place of two
// launches that move every pair through memory; sorted pairs, bags and sums are those of the partitioned path, bit for
// bit.  Bound by the chain of latencies: row ids, sort, offsets, gradient and table rows.
template <int DT, int G, int OPT, bool WT, bool KEEP>
__global__ __launch_bounds__(kThreads, (OPT == kAdagrad || DT == DLRM_F32) ? 3 : 4) void direct_reduce_kernel(GroupArgs a, UpdArgs u) {
  __shared__ SortLds s;
  __shared__ SplitLds sp;
  __shared__ float part[kThreads * 4];
  __shared__ float wext[WT ? kBktCap - kResolvedLo : 1];
  const int tid = threadIdx.x;
  const uint32_t id = blockIdx.x;
  Bucket b;
  b.k = (int)(id >> a.top_bits);
  const uint32_t dg = id & ((1u << a.top_bits) - 1u);
  if (tid == 0 && id == 0) a.seg_meta[kRouteDirect] = 1u;
  b.route = a.hist + (size_t)id * kRouteWords;   // this workgroup's own counters
  if (tid < kRouteWords) b.route[tid] = 0u;
  const int64_t tbl = a.tbl_off[b.k];
  const uint32_t nk = (uint32_t)(a.tbl_off[b.k + 1] - tbl);
  const int shift = top_shift(a, b.k);
  char* W = static_cast<char*>(u.tables[b.k]);
  b.H = state_base<OPT>(u, b.k);
  if (nk == 0 || ((int64_t)dg << shift) >= a.rows[b.k]) return;
  BagSearch bags;
  bags.off = a.offsets + (int64_t)b.k * (a.B + 1);
  bags.B = (uint32_t)a.B;
  bags.step = 1;
  while (bags.step * kThreads < bags.B) bags.step <<= 1;
  bags.nsmp = (bags.B + bags.step - 1) / bags.step;
  bags.fixed = nk % bags.B == 0 ? nk / bags.B : 0u;
  bags.smp = s.heads;
  if ((uint32_t)tid < bags.nsmp) s.heads[tid] = (uint32_t)bags.off[(uint32_t)tid * bags.step];
  const int32_t* const idx4 = static_cast<const int32_t*>(a.indices) + tbl;
  const int64_t* const idx8 = static_cast<const int64_t*>(a.indices) + tbl;
  unsigned long long* const mask = reinterpret_cast<unsigned long long*>(s.skey);
  uint32_t less = 0, before = 0;
  if (nk <= (uint32_t)kBktCap) {   // uniform
    b.n = a.idx32 ? pick_lookups(idx4, nk, dg, shift, s) : pick_lookups(idx8, nk, dg, shift, s);
  } else {
    less = a.idx32 ? mark_lookups(idx4, nk, dg, shift, mask) : mark_lookups(idx8, nk, dg, shift, mask);
    __syncthreads();
    before = block_exclusive_scan<kThreads>(count_marked(mask, nk), s.smem, &b.n);
  }
  b.n = uniform(b.n);
  b.low_bits = shift;
  b.start = 0;
  if (b.n == 0) return;
  if (tid == 0 && b.n > a.big) b.route[kRouteHeavy] = 1u;
  const ResolvedW rw{reinterpret_cast<float*>(&s.wcnt[0][0]), wext};
  if (b.n <= (uint32_t)kBktCap) {
    if (nk > (uint32_t)kBktCap) {   // uniform
      marked_positions(mask, nk, before, [&](uint32_t i, uint32_t pos) { s.sval[i] = pos; });
      __syncthreads();
      if (a.idx32)
        rows_of_positions(idx4, s.sval, b.n, s.skey);
      else
        rows_of_positions(idx8, s.sval, b.n, s.skey);
    }
    __syncthreads();
    sort_bucket_lds<true>(a, b, s);
    uint32_t pos[kBktItems], bag[kBktItems];
    float ew[WT ? kBktItems : 1];
#pragma unroll
    for (int j = 0; j < kBktItems; ++j) {
      const uint32_t li = tid + j * kThreads;
      pos[j] = s.sval[li < b.n ? li : 0];
    }
    __syncthreads();   // sval[0] may be read by every thread, and its owner rewrites it below
    if constexpr (WT) {
#pragma unroll
      for (int j = 0; j < kBktItems; ++j) ew[j] = a.weights[tbl + pos[j]];
    }
    if (b.n <= (uint32_t)(2 * kThreads)) {
      bags.find_all<2>(pos, bag);
    } else {
      bags.find_all<kBktItems>(pos, bag);
    }
#pragma unroll
    for (int j = 0; j < kBktItems; ++j) {  // a thread rewrites only the slots it read
      const uint32_t li = tid + j * kThreads;
      if (li < b.n) {
        s.sval[li] = bag[j];
        if constexpr (WT) rw.at(li) = ew[j];
      }
    }
    __syncthreads();
    reduce_slabs<DT, G, OPT, WT, KEEP>(u, b, W, s.skey, s.sval, b.n, part, s.heads, rw);
    return;
  }
  // too many pairs for the LDS sort: the bucket is laid out in pair buffer 1 as the partition would
  if (tid == 0) b.route[kRouteOver] = 1u;
  {
    uint32_t all;
    block_exclusive_scan<kThreads>(lane_id() == 0 ? less : 0u, s.smem, &all);
    b.start = uniform((uint32_t)tbl + all);
  }
  uint32_t* kout = a.keys[1] + b.start;
  uint32_t* vout = a.vals[1] + b.start;
  marked_positions(mask, nk, before, [&](uint32_t i, uint32_t pos) { vout[i] = pos; });
  __syncthreads();
  if (a.idx32)
    rows_of_positions(idx4, vout, b.n, kout);
  else
    rows_of_positions(idx8, vout, b.n, kout);
  constexpr int N = kBktItems / 2;
  for (uint32_t i0 = 0; i0 < b.n; i0 += N * kThreads) {   // positions -> bags (weighted: bags and weights beside them)
    uint32_t pos[N], bag[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const uint32_t i = i0 + tid + j * kThreads;
      pos[j] = vout[i < b.n ? i : b.n - 1];
    }
    if (i0 + N * kThreads >= b.n) __syncthreads();   // uniform: the last entry has been read by all before its owner rewrites it
    bags.find_all<N>(pos, bag);
    if constexpr (WT) {
      float w[N];
#pragma unroll
      for (int j = 0; j < N; ++j) w[j] = a.weights[tbl + pos[j]];
#pragma unroll
      for (int j = 0; j < N; ++j)
        if (i0 + tid + j * kThreads < b.n) a.pos_entry[tbl + pos[j]] = PosEntry{bag[j], w[j]};
    } else {
#pragma unroll
      for (int j = 0; j < N; ++j)
        if (i0 + tid + j * kThreads < b.n) vout[i0 + tid + j * kThreads] = bag[j];
    }
  }
  __syncthreads();
  reduce_beyond_lds<DT, G, OPT, WT>(a, u, b, W, s, sp, part, rw);
}

template <int DT, int G, int OPT, bool WT>
__global__ __launch_bounds__(kThreads) void segment_reduce_kernel(GroupArgs a, UpdArgs u) {
  __shared__ SortLds s;
  __shared__ float part[kThreads * 4];
  SegInfo sg;
  uint32_t t;
  if (!find_segment_tile(a, &sg, &t)) return;
  Bucket b;
  b.k = (int)sg.k;
  b.start = sg.start;
  b.n = sg.n;
  b.low_bits = 0;
  b.route = a.seg_meta;
  b.H = state_base<OPT>(u, b.k);
  char* W = static_cast<char*>(u.tables[b.k]);
  const int dst = (int)(sg.src ^ 1u);
  reduce_window<DT, G, OPT, WT>(a, u, b, W, a.keys[dst] + sg.start, a.vals[dst] + sg.start, t * kBktCap, dst, s, part);
}


template <int DT, int G, int OPT, bool WT, bool KEEP>
static void launch_buckets(const GroupArgs& g, const UpdArgs& u, int K, hipStream_t st) {
  const unsigned buckets = (unsigned)K << g.top_bits;
  if (g.direct)
    hipLaunchKernelGGL((direct_reduce_kernel<DT, G, OPT, WT, KEEP>), dim3(buckets), dim3(kThreads), 0, st, g, u);
  else
    hipLaunchKernelGGL((bucket_reduce_kernel<DT, G, OPT, WT, KEEP>), dim3(buckets + (unsigned)g.max_over), dim3(kThreads),
                       0, st, g, u);
}

template <int DT, int G, int OPT, bool WT>
static int launch_reduce(const GroupArgs& g, const UpdArgs& u, int K, const dlrm_bwd_timing* tm, hipStream_t st) {
  if (tm && tm->ev_start && hipEventRecord(static_cast<hipEvent_t>(tm->ev_start), st) != hipSuccess) return DLRM_ERR_HIP;
  constexpr int narrowest = (G > 1 ? 2 * G + 4 : 4) * Tab<DT>::EB;   // bytes of the narrowest row of G lanes
  if constexpr (narrowest < keep_below(DT, OPT)) {
    if (rows_share_sectors(u.d, DT, OPT))
      launch_buckets<DT, G, OPT, WT, true>(g, u, K, st);
    else
      launch_buckets<DT, G, OPT, WT, false>(g, u, K, st);
  } else {
    launch_buckets<DT, G, OPT, WT, false>(g, u, K, st);
  }
  DLRM_CHECK_LAUNCH();
  if (tm && tm->ev_stop && hipEventRecord(static_cast<hipEvent_t>(tm->ev_stop), st) != hipSuccess) return DLRM_ERR_HIP;
  if (g.no_tail) return DLRM_OK;
  const unsigned seg_tiles = (unsigned)(g.seg_tiles_max);
  int rc = launch_segment_sort(g, st);
  if (rc != DLRM_OK) return rc;
  hipLaunchKernelGGL((segment_reduce_kernel<DT, G, OPT, WT>), dim3(seg_tiles), dim3(kThreads), 0, st, g, u);
  DLRM_CHECK_LAUNCH();
  return launch_hot_rows(g, u, G, DT, OPT, st);
}

template <int DT, int OPT, bool WT>
static int dispatch_reduce(const GroupArgs& g, const UpdArgs& u, int G, int K, const dlrm_bwd_timing* tm, hipStream_t st) {
  switch (G) {
    case 1: return launch_reduce<DT, 1, OPT, WT>(g, u, K, tm, st);
    case 2: return launch_reduce<DT, 2, OPT, WT>(g, u, K, tm, st);
    case 4: return launch_reduce<DT, 4, OPT, WT>(g, u, K, tm, st);
    case 8: return launch_reduce<DT, 8, OPT, WT>(g, u, K, tm, st);
    case 16: return launch_reduce<DT, 16, OPT, WT>(g, u, K, tm, st);
    case 32: return launch_reduce<DT, 32, OPT, WT>(g, u, K, tm, st);
    case 64: return launch_reduce<DT, 64, OPT, WT>(g, u, K, tm, st);
  }
  return DLRM_ERR_BAD_SHAPE;
}


template <int OPT, bool WT>
inline int run_reduce(const GroupArgs& g, const UpdArgs& u, int dtype, int G, int K, const dlrm_bwd_timing* tm, hipStream_t st) {
  switch (dtype) {
    case DLRM_F32: return dispatch_reduce<DLRM_F32, OPT, WT>(g, u, G, K, tm, st);
    case DLRM_F16: return dispatch_reduce<DLRM_F16, OPT, WT>(g, u, G, K, tm, st);
    case DLRM_BF16: return dispatch_reduce<DLRM_BF16, OPT, WT>(g, u, G, K, tm, st);
  }
  return DLRM_ERR_BAD_DTYPE;
}

}  // namespace dlrm
