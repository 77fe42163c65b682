// Dot-product feature interaction (Sec. 2.2) and its backward.
//   fwd: R[b] = [ T[b,0,:] | <T[b,i,:],T[b,j,:]> for 1 <= i < F, 0 <= j < i ]
//   bwd: dT[b,i,:] = sum_{j != i} g(i,j) T[b,j,:]  (+ dR[b,0:d] on row 0),
//        g(i,j) = dR[b, d + pair(max(i,j), min(i,j))]
// Both are small dense contractions per sample (Z = T T^t, dT = G T with G symmetric), run on
// the matrix cores in fp32: v_mfma_f32_16x16x4_f32.  A wavefront per sample loads its operands
// straight from global memory into the register layout the instruction wants (no LDS staging
// of T, no workgroup barriers), so HBM sees each input and output once.  A workgroup per sample
// takes over where one wavefront is a long chain or too few fit a compute unit: the forward from
// three row blocks on stages T in LDS (interact_fwd_split_kernel, split_fwd), the backward lays
// out G there (interact_bwd_tiled_kernel, kSplitBelow); both with barriers and with the same bits.
//   16x16x4 layout: lane l supplies A[m = l%16][k = l/16] and B[k = l/16][n = l%16] and holds
//   D[m = 4*(l/16) + v][n = l%16] in element v of its accumulator.
// The contraction index may be visited in any order as long as A and B agree on it, which is
// what lets every lane fetch 16 contiguous bytes and use them in 4 consecutive instructions.
#include "common.h"

#include <type_traits>

namespace dlrm {

constexpr int kIntThreads = 256;
constexpr int kIntWaves = kIntThreads / DLRM_WAVE;   // samples per workgroup

__device__ inline f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// --- forward --------------------------------------------------------------------------------
// Row 0 of T_b (the dense vector) is kept apart; the K = F-1 embedding rows form NB blocks of
// 16.  Lane (i = l%16, h = l/16) fetches, for every row block, the 4 floats at columns 16q + 4h
// of embedding row 16*rb + i.  Element t of that float4 is at once the A operand of the row
// block and the B operand of the column block for the 4 columns {16q + 4h' + t : h' = 0..3},
// so a tile (ib, jb) of Z = S S^t takes one instruction per 4 columns; only tiles on or below
// the diagonal are computed.  The K products with the dense row are plain FMAs on the same
// registers (a 17th row would cost a whole extra row and column of tiles).
template <int NB>
__global__ __launch_bounds__(kIntThreads) void interact_fwd_kernel(const float* __restrict__ T,
                                                                    float* __restrict__ R, int B, int F,
                                                                    int d, int pstride) {
  constexpr int QC = NB <= 2 ? 4 : 2;  // 16-column chunks fetched per round
  constexpr int NTILE = NB * (NB + 1) / 2;
  extern __shared__ float lds[];
  const int lane = lane_id();
  const int b = blockIdx.x * kIntWaves + wave_id();
  if (b >= B) return;  // wavefronts are independent: no barriers below
  const int i = lane & 15, h = lane >> 4;
  const int K = F - 1;
  const int P = F * (F - 1) / 2;
  const float* Tb = T + (int64_t)b * F * d;
  float* Rb = R + (int64_t)b * ((int64_t)d + P);
  f32x4 acc[NTILE];
#pragma unroll
  for (int t = 0; t < NTILE; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const float* rowp[NB];
  float pd[NB];  // partial products with the dense row
#pragma unroll
  for (int rb = 0; rb < NB; ++rb) {
    // rows past the last one repeat it (the dense row if there is none): their products land in
    // entries that are never stored
    const int e = rb * 16 + i < K ? rb * 16 + i : K - 1;
    rowp[rb] = Tb + (int64_t)(e + 1) * d;
    pd[rb] = 0.0f;
  }
  for (int k0 = 0; k0 < d; k0 += 16 * QC) {
    f32x4 x0[QC], x[NB][QC];
#pragma unroll
    for (int q = 0; q < QC; ++q) {
      const int col = k0 + 16 * q + 4 * h;
      const int ccol = col < d ? col : 0;
      const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
      const f32x4 v0 = loadf4(Tb + ccol);
      x0[q] = col < d ? v0 : zero;
#pragma unroll
      for (int rb = 0; rb < NB; ++rb) {
        const f32x4 v = loadf4(rowp[rb] + ccol);
        x[rb][q] = col < d ? v : zero;  // columns past d contribute 0 * 0
      }
    }
#pragma unroll
    for (int q = 0; q < QC; ++q) {
      if (k0 + 16 * q < d) {  // uniform
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) {
          pd[rb] = fmaf(x[rb][q].x, x0[q].x, pd[rb]);
          pd[rb] = fmaf(x[rb][q].y, x0[q].y, pd[rb]);
          pd[rb] = fmaf(x[rb][q].z, x0[q].z, pd[rb]);
          pd[rb] = fmaf(x[rb][q].w, x0[q].w, pd[rb]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          int tile = 0;
#pragma unroll
          for (int ib = 0; ib < NB; ++ib) {
#pragma unroll
            for (int jb = 0; jb <= ib; ++jb, ++tile) acc[tile] = mfma16(x[ib][q][t], x[jb][q][t], acc[tile]);
          }
        }
      }
    }
  }
  // The accumulator layout scatters the pairs; they are gathered in this wavefront's LDS and
  // leave as whole contiguous lines (partial-line writes cost a fill read each).
  float* Rp = lds + wave_id() * pstride;
  // pair (gi, gj), gi > gj, sits at gi(gi-1)/2 + gj; embedding row e is row e + 1 of T
#pragma unroll
  for (int rb = 0; rb < NB; ++rb) {
    float v = pd[rb];
    v += __shfl_xor(v, 16, DLRM_WAVE);
    v += __shfl_xor(v, 32, DLRM_WAVE);
    const int e = rb * 16 + i;
    if (h == 0 && e < K) Rp[(e + 1) * e / 2] = v;
  }
  int tile = 0;
#pragma unroll
  for (int ib = 0; ib < NB; ++ib) {
#pragma unroll
    for (int jb = 0; jb <= ib; ++jb, ++tile) {
      const int ej = jb * 16 + i;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ei = ib * 16 + 4 * h + v;
        if (ej < ei && ei < K) Rp[(ei + 1) * ei / 2 + ej + 1] = acc[tile][v];
      }
    }
  }
  for (int c = lane; c < d; c += DLRM_WAVE) Rb[c] = Tb[c];  // dense part: exact copy of row 0
  for (int c = lane; c < P; c += DLRM_WAVE) Rb[d + c] = Rp[c];
}

// The same products, instructions and order with a workgroup of W wavefronts per sample (W <= NB <= 2 W) and T_b staged in LDS,
// kSplitCols columns at a time: each row is read from memory once, along its columns, where the operand layout reads 64 bytes
// of 16 rows at a time.  Wavefront w computes the tiles of row blocks NB - 1 - w and, where there is one, w - (2 W - NB), which
// deals the tiles evenly (seven blocks: seven each), and the dense row's products with them; all leave together.  Bound by the
// chain of one sample at small batches, by memory at large ones (65 rows of 128 columns, batch 16384: 4.5 of the copy's 4.6 TB/s).
// Three wavefronts per SIMD up to seven row blocks.  Eight would have 26 registers spilled by that, between the staged columns of
// rows wider than kSplitCols; those have two.  A wavefront per sample / three to a SIMD / two, us: 128 rows of 256 columns, batch 1024 /
// 4096 64.1 / 81.8 / 57.1, 263.5 / 284.5 / 210.5; of 96, 4096 135.7 / 147.5 / 110.5.  Rows of one stage have a kernel of their own
// without the loop: no row waits in registers while others are multiplied, 84 of them, and the LDS sets the limit.  With the loop, three to
// a SIMD / its own: 125 rows of 28, batch 506 11.2 / 9.7; 122 of 4, 5032 54.3 / 38.0; 128 of 64, 1257 30.7 / 27.9.  Operands read
// from memory by each of the four wavefronts instead of from LDS: 101 rows of 64, batch 16384 377 us for 209.7.
constexpr int kSplitCols = 64;
// words of a staged row: whole 16-column chunks, and 4 words so that the 16 rows an operand is read from fall into 64 banks
__host__ __device__ inline int split_stride(int d) { return (d < kSplitCols ? (d + 15) & ~15 : kSplitCols) + 4; }
template <int NB, int W>
constexpr int kSplitTiles = NB > 2 * NB - 2 * W + 1 ? NB : 2 * NB - 2 * W + 1;   // of a wavefront, at most

// Wavefront w's tiles, one after the other: of row block I1, then of row block I0.  lo: the lane's place in the first staged
// embedding row.
template <int NB, int W, int w>
struct SplitShare {
  static constexpr int I1 = NB - 1 - w, I0 = w - (2 * W - NB), N1 = I1 + 1, N0 = I0 < 0 ? 0 : I0 + 1;
  static_assert(N1 + N0 <= kSplitTiles<NB, W>, "a register for each");
  // the 16-column chunks of the staged columns, `cols` of them
  static __device__ inline void products(const float* lo, int cs, int cols, f32x4* acc, float* pd) {
#pragma unroll
    for (int q = 0; q < kSplitCols / 16; ++q) {
      if (16 * q < cols) {  // uniform
        const f32x4 xd = loadf4(lo + 16 * q - (int)(threadIdx.x & 15) * cs - cs);   // the dense row
        f32x4 x[NB];
#pragma unroll
        for (int jb = 0; jb <= I1; ++jb) x[jb] = loadf4(lo + jb * 16 * cs + 16 * q);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          pd[0] = fmaf(x[I1][t], xd[t], pd[0]);
          if constexpr (N0 > 0) pd[1] = fmaf(x[I0][t], xd[t], pd[1]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
          for (int jb = 0; jb < N1; ++jb) acc[jb] = mfma16(x[I1][t], x[jb][t], acc[jb]);
#pragma unroll
          for (int jb = 0; jb < N0; ++jb) acc[N1 + jb] = mfma16(x[N0 > 0 ? I0 : 0][t], x[jb][t], acc[N1 + jb]);
        }
      }
    }
  }
  template <int ib>
  static __device__ inline void put_row_block(float* pairs, int K, const f32x4* acc, float v) {
    const int i = lane_id() & 15, h = lane_id() >> 4;
    v += __shfl_xor(v, 16, DLRM_WAVE);
    v += __shfl_xor(v, 32, DLRM_WAVE);
    const int e = ib * 16 + i;
    if (h == 0 && e < K) pairs[(e + 1) * e / 2] = v;
#pragma unroll
    for (int jb = 0; jb <= ib; ++jb) {
      const int ej = jb * 16 + i;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int ei = ib * 16 + 4 * h + c;
        if (ej < ei && ei < K) pairs[(ei + 1) * ei / 2 + ej + 1] = acc[jb][c];
      }
    }
  }
  static __device__ inline void put(float* pairs, int K, const f32x4* acc, const float* pd) {
    put_row_block<I1>(pairs, K, acc, pd[0]);
    if constexpr (N0 > 0) put_row_block<I0>(pairs, K, acc + N1, pd[1]);
  }
};
// f(SplitShare of this wavefront)
template <int NB, int W, typename F>
__device__ inline void for_share(int w, F f) {
  if (w == 0) f(SplitShare<NB, W, 0>());
  if (w == 1) f(SplitShare<NB, W, 1>());
  if constexpr (W > 2) {
    if (w == 2) f(SplitShare<NB, W, 2>());
    if (w == 3) f(SplitShare<NB, W, 3>());
  }
}

template <int NB, int W, bool WIDE>   // WIDE: rows of more than kSplitCols columns too
__global__ __launch_bounds__(W * DLRM_WAVE, NB == 8 && WIDE ? 2 : 3) void interact_fwd_split_kernel(const float* __restrict__ T,
                                                                                                  float* __restrict__ R, int F,
                                                                                                  int d) {
  static_assert(W <= NB && NB <= 2 * W && (W == 2 || W == 4), "one or two row blocks a wavefront");
  constexpr int NT = W * DLRM_WAVE;
  constexpr int RP = NT / 16;                       // rows staged per pass, 16 bytes a lane
  constexpr int NP = (16 * NB + 1 + RP - 1) / RP;   // passes
  extern __shared__ __align__(16) float lds[];
  const int lane = lane_id(), w = (int)__builtin_amdgcn_readfirstlane(wave_id());
  const int tl = w * DLRM_WAVE + lane;
  const int b = blockIdx.x;
  const int K = F - 1;
  const int P = F * (F - 1) / 2;
  const float* Tb = T + (int64_t)b * F * d;
  float* Rb = R + (int64_t)b * ((int64_t)d + P);
  const int cs = split_stride(d);
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 acc[kSplitTiles<NB, W>];
#pragma unroll
  for (int t = 0; t < kSplitTiles<NB, W>; ++t) acc[t] = zero;
  float pd[2] = {0.0f, 0.0f};   // partial products with the dense row
  const int srow = tl >> 4, scol = 4 * (tl & 15);   // this thread's piece of a pass
  f32x4 v[NP];
  const auto request = [&](int k0) {   // (rows past the last one and columns past d repeat others: no load behind a branch)
    const int col = k0 + scol < d ? k0 + scol : 0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int r = p * RP + srow < F ? p * RP + srow : F - 1;
      v[p] = loadf4(Tb + (int64_t)r * d + col);
    }
  };
  request(0);
  // row e + 1 of T_b is embedding row e; operands of rows past the last one are whatever lies there: their products land in
  // entries that are never stored
  const float* const lo = lds + ((lane & 15) + 1) * cs + 4 * (lane >> 4);
  for (int k0 = 0; k0 < d; k0 += kSplitCols) {
    if (k0 > 0) __syncthreads();   // the previous columns have been read
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int r = p * RP + srow;
      if (r < F && scol + 4 < cs) storef4(lds + r * cs + scol, k0 + scol < d ? v[p] : zero);   // columns past d contribute 0 * 0
    }
    __syncthreads();
    if constexpr (WIDE) {
      if (k0 + kSplitCols < d) request(k0 + kSplitCols);   // on their way while these are multiplied
    }
    for_share<NB, W>(w, [&](auto share) { share.products(lo, cs, d - k0, acc, pd); });
    if constexpr (!WIDE) break;
  }
  for (int c = tl; c < d; c += NT) Rb[c] = Tb[c];  // dense part: exact copy of row 0
  __syncthreads();   // the staged rows have been read: the pairs take their place
  for_share<NB, W>(w, [&](auto share) { share.put(lds, K, acc, pd); });
  __syncthreads();
  for (int c0 = 0; c0 < P; c0 += NT * 8) {
    float r[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int c = c0 + q * NT + tl;
      r[q] = lds[c < P ? c : P - 1];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int c = c0 + q * NT + tl;
      if (c < P) Rb[d + c] = r[q];
    }
  }
}

// --- backward -------------------------------------------------------------------------------
// dT_b = G T_b with G the symmetric F x F matrix of pair gradients (zero diagonal), held per
// wavefront in LDS as the lower triangle exactly as dR stores it.  For the K embedding rows,
// row block ib of G is the A operand (lane: embedding row 16*ib + l%16, column 4s + l/16 in
// step s); the B operand of step s is embedding row 4s + l/16, of which lane x = l%16 fetches
// CW = 4, 2 or 1 floats at columns 16*CW*g + CW*x: element u of them belongs to the output tile
// whose 16 columns are {16*CW*g + CW*x' + u}, so that after the contraction every lane owns CW
// consecutive columns of 4 rows and stores them as one vector.  The dense row enters and leaves through plain FMAs: a rank-1
// update of every tile, and one matrix-vector product for its own gradient.
template <int NB, int CW>
__global__ __launch_bounds__(kIntThreads) void interact_bwd_kernel(const float* __restrict__ T,
                                                                    const float* __restrict__ dR,
                                                                    float* __restrict__ dT, int B, int F,
                                                                    int d, int gstride) {
  constexpr int JS = 4 * NB;  // contraction steps of 4 embedding rows
  extern __shared__ float lds[];
  const int lane = lane_id();
  const int b = blockIdx.x * kIntWaves + wave_id();
  if (b >= B) return;  // wavefronts are independent: no barriers below
  const int x_ = lane & 15, h_ = lane >> 4;
  const int K = F - 1;
  const int P = F * (F - 1) / 2;
  const float* Tb = T + (int64_t)b * F * d;
  const float* gR = dR + (int64_t)b * ((int64_t)d + P);
  float* dTb = dT + (int64_t)b * F * d;
  float* gs = lds + wave_id() * gstride;
  for (int t0 = 0; t0 < P; t0 += DLRM_WAVE * 16) {  // 16 loads in flight per lane
    float v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int idx = t0 + q * DLRM_WAVE + lane;
      v[q] = gR[d + (idx < P ? idx : P - 1)];
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int idx = t0 + q * DLRM_WAVE + lane;
      if (idx < P) gs[idx] = v[q];
    }
  }
  for (int g0 = 0; g0 < d; g0 += 16 * CW) {
    // opaque copies: without them every row offset, LDS index and validity mask below is
    // hoisted out of this loop and held in registers, which halves the occupancy
    int x = x_, h = h_;
    asm volatile("" : "+v"(x), "+v"(h));
    const int col = g0 + CW * x;
    const bool cok = col < d;
    const int ccol = cok ? col : 0;
    float tb[JS][CW], t0v[CW];
    load_cols<CW>(Tb + ccol, cok, t0v);
#pragma unroll
    for (int s = 0; s < JS; ++s) {
      const int e = 4 * s + h;
      load_cols<CW>(Tb + (int64_t)((e < K ? e : K - 1) + 1) * d + ccol, e < K && cok, tb[s]);
    }
    // gradient of the dense row: dR[0:d] + sum_e g(e+1, 0) S_e; g(e+1, 0) sits at (e+1)e/2
    {
      float a0[CW];
#pragma unroll
      for (int c = 0; c < CW; ++c) a0[c] = 0.0f;
#pragma unroll
      for (int s = 0; s < JS; ++s) {
        const int e = 4 * s + h;
        const float gv = gs[e < K ? (e + 1) * e / 2 : 0];
        const float g0e = e < K ? gv : 0.0f;
#pragma unroll
        for (int c = 0; c < CW; ++c) a0[c] = fmaf(g0e, tb[s][c], a0[c]);
      }
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        a0[c] += __shfl_xor(a0[c], 16, DLRM_WAVE);
        a0[c] += __shfl_xor(a0[c], 32, DLRM_WAVE);
      }
      if (h == 0 && cok) {
#pragma unroll
        for (int c = 0; c < CW; ++c) a0[c] += gR[col + c];
        store_cols<CW>(dTb + col, a0);
      }
    }
#pragma unroll(NB <= 2 ? NB : 1)
    for (int ib = 0; ib < NB; ++ib) {  // many row blocks: one at a time keeps the register count down
      if (ib * 16 >= K) break;  // uniform
      const int m = ib * 16 + x;
      float ga[JS];
#pragma unroll
      for (int s = 0; s < JS; ++s) {
        const int e = 4 * s + h;
        const int hi = m > e ? m : e, lo = m > e ? e : m;
        const bool ok = hi < K && hi != lo;
        const float gv = gs[ok ? (hi + 1) * hi / 2 + lo + 1 : 0];
        ga[s] = ok ? gv : 0.0f;
      }
      float gd[4];  // g(row, 0) of this lane's 4 output rows
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ei = ib * 16 + 4 * h + v;
        const float gv = gs[ei < K ? (ei + 1) * ei / 2 : 0];
        gd[v] = ei < K ? gv : 0.0f;
      }
      f32x4 acc[CW];
#pragma unroll
      for (int u = 0; u < CW; ++u) acc[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < JS; ++s) {
        if (4 * s < K) {  // uniform
#pragma unroll
          for (int u = 0; u < CW; ++u) acc[u] = mfma16(ga[s], tb[s][u], acc[u]);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ei = ib * 16 + 4 * h + v;
        if (ei < K && cok) {
          float o[CW];
#pragma unroll
          for (int u = 0; u < CW; ++u) o[u] = fmaf(gd[v], t0v[u], acc[u][v]);
          store_cols<CW>(dTb + (int64_t)(ei + 1) * d + col, o);
        }
      }
    }
  }
}

// The same contraction, instructions and order with a workgroup of WPS wavefronts per sample: they share one copy of G
// and take every WPS-th row block each; the last one, which never has more blocks, adds the dense row.
// G lies in LDS as the 16 x 16 tiles on and below the diagonal of its embedding part (rows of 17 words; the diagonal
// tiles whole, rows past the last one zero) and its dense column: the A operand of (ib, step s) is one word per lane at
// a lane offset plus a constant, read along or across a tile, where the triangle as dR stores it costs a dozen address
// instructions per operand.  dR is fetched in 16-byte pieces, all in flight at once.
// Taken from six row blocks on (a wavefront per sample there: one wavefront per SIMD, a copy of G each), with five by
// batch and columns (kSplitBelow5), and with fewer up to kSplitBelow samples (SIMDs with one wavefront or none): 101 rows
// of 64 columns, batch 64 / 1024 / 8192: 54.7 / 60.8 / 295 us with a wavefront per sample, 17.2 / 39.3 / 260 us here; 65
// rows of 128: 31.7 / 38.6 / 171 and 11.1 / 28.1 / 182 us; 27 rows of 64: 6.1 / 7.2 / 28.5 and 4.7 / 6.3 / 30.4 us.
// Bound by the chain of one sample at small batches (101 rows of 32 columns, batch 1024: matrix cores busy 16 % of 28 us);
// at large ones the matrix cores, 700 instructions of 32 cycles a sample, are busy for 75 of the 260 us.
constexpr int kGRow = 17, kGTile = 16 * kGRow;
__host__ __device__ constexpr int g_words(int NB) { return NB * (NB + 1) / 2 * kGTile + 16 * NB; }

template <int NB, int WPS, int CW>
__global__ __launch_bounds__(WPS * DLRM_WAVE) void interact_bwd_tiled_kernel(
    const float* __restrict__ T, const float* __restrict__ dR, float* __restrict__ dT, int F, int d) {
  constexpr int JS = 4 * NB;  // contraction steps of 4 embedding rows
  extern __shared__ __align__(16) float lds[];
  const int lane = lane_id();
  const int sub = wave_id();
  const int b = blockIdx.x;
  const int x_ = lane & 15, h_ = lane >> 4;
  const int K = F - 1;
  const int P = F * (F - 1) / 2;
  const float* Tb = T + (int64_t)b * F * d;
  const float* gR = dR + (int64_t)b * ((int64_t)d + P);
  float* dTb = dT + (int64_t)b * F * d;
  float* gs = lds;
  float* gd0 = gs + NB * (NB + 1) / 2 * kGTile;   // g(e + 1, 0)
  constexpr int NT = WPS * DLRM_WAVE;
  const int tl = sub * DLRM_WAVE + lane;
  // pair gradients in 16-byte pieces (dR's rows start anywhere), all requested before anything is waited for;
  // the pieces that would reach past the sample's last pair are left to single loads
  const float* gP = gR + d;
  const int mis = (int)((reinterpret_cast<uintptr_t>(gP) >> 2) & 3);
  const float* gA = gP - mis;   // aligned; at most 3 words back, which the dense part of dR holds
  const int nq = (P + mis) >> 2;
  constexpr int GL = ((16 * NB + 1) * 16 * NB / 8 + NT) / NT;   // pieces per lane
  f32x4 v[GL];
#pragma unroll
  for (int q = 0; q < GL; ++q) {
    const int t = q * NT + tl;
    v[q] = loadf4(gA + (t < nq ? t : 0) * 4);
  }
  const int tail = nq * 4 - mis + tl;
  const float vt = tail < P ? gP[tail < 0 ? 0 : tail] : 0.0f;
  // pair (i, j), i > j, sits at i(i-1)/2 + j; as embedding rows: (i - 1, j - 1), j = 0 the dense row
  auto put = [&](int e, int f, float val) {
    const int I = e >> 4, J = f >> 4;
    const int r = e & 15, c = f & 15;
    float* tile = gs + (I * (I + 1) / 2 + J) * kGTile;
    if (f < 0) {
      gd0[e] = val;
    } else {
      tile[r * kGRow + c] = val;
      if (I == J) tile[c * kGRow + r] = val;
    }
  };
  auto row_of = [](int idx) {
    int i = (int)((1.0f + sqrtf((float)(8 * idx + 1))) * 0.5f);
    i -= i * (i - 1) / 2 > idx ? 1 : 0;
    i += i * (i + 1) / 2 <= idx ? 1 : 0;
    return i;
  };
  float tb[JS][CW], t0v[CW];
  auto load_rows = [&](int x, int h, int g0) {
    const int col = g0 + CW * x;
    const bool cok = col < d;
    const int ccol = cok ? col : 0;
    load_cols<CW>(Tb + ccol, cok, t0v);
#pragma unroll
    for (int s = 0; s < JS; ++s) {
      const int e = 4 * s + h;
      load_cols<CW>(Tb + (int64_t)((e < K ? e : K - 1) + 1) * d + ccol, e < K && cok, tb[s]);
    }
  };
  for (int t = tl * 4; t < g_words(NB); t += NT * 4) storef4(gs + t, f32x4{0.0f, 0.0f, 0.0f, 0.0f});
  __syncthreads();
#pragma unroll
  for (int q = 0; q < GL; ++q) {
    const int t = q * NT + tl, first = 4 * t - mis;
    if (t >= nq) continue;
    int i = row_of(first < 0 ? 0 : first), jj = (first < 0 ? 0 : first) - i * (i - 1) / 2;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (first + c < 0) continue;
      put(i - 1, jj - 1, v[q][c]);
      if (++jj == i) {
        ++i;
        jj = 0;
      }
    }
  }
  if (tail >= 0 && tail < P && tl < 4) {
    const int i = row_of(tail);
    put(i - 1, tail - i * (i - 1) / 2 - 1, vt);
  }
  load_rows(x_, h_, 0);
  __syncthreads();
  for (int g0 = 0; g0 < d; g0 += 16 * CW) {
    // opaque copies: without them every row offset, LDS index and validity mask below is
    // hoisted out of this loop and held in registers, which halves the occupancy
    int x = x_, h = h_;
    asm volatile("" : "+v"(x), "+v"(h));
    const int col = g0 + CW * x;
    const bool cok = col < d;
    if (g0 > 0) load_rows(x, h, g0);
    // gradient of the dense row: dR[0:d] + sum_e g(e+1, 0) S_e
    if (sub == WPS - 1) {   // uniform
      float a0[CW];
#pragma unroll
      for (int c = 0; c < CW; ++c) a0[c] = 0.0f;
#pragma unroll
      for (int s = 0; s < JS; ++s) {
        const float g0e = gd0[4 * s + h];
#pragma unroll
        for (int c = 0; c < CW; ++c) a0[c] = fmaf(g0e, tb[s][c], a0[c]);
      }
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        a0[c] += __shfl_xor(a0[c], 16, DLRM_WAVE);
        a0[c] += __shfl_xor(a0[c], 32, DLRM_WAVE);
      }
      if (h == 0 && cok) {
#pragma unroll
        for (int c = 0; c < CW; ++c) a0[c] += gR[col + c];
        store_cols<CW>(dTb + col, a0);
      }
    }
    const float* along = gs + x * kGRow + h;
    const float* across = gs + h * kGRow + x;
#pragma unroll 1
    for (int ib = sub; ib < NB; ib += WPS) {  // one row block at a time keeps the register count down
      if (ib * 16 >= K) break;  // uniform
      float ga[JS];
#pragma unroll
      for (int J = 0; J < NB; ++J) {
        if (J <= ib) {  // uniform
          const float* t = along + (ib * (ib + 1) / 2 + J) * kGTile;
#pragma unroll
          for (int q = 0; q < 4; ++q) ga[4 * J + q] = t[4 * q];
        } else {
          const float* t = across + (J * (J + 1) / 2 + ib) * kGTile;
#pragma unroll
          for (int q = 0; q < 4; ++q) ga[4 * J + q] = t[4 * q * kGRow];
        }
      }
      const f32x4 gd = loadf4(gd0 + ib * 16 + 4 * h);   // g(row, 0) of this lane's 4 output rows
      f32x4 acc[CW];
#pragma unroll
      for (int u = 0; u < CW; ++u) acc[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < JS; ++s) {
        if (4 * s < K) {  // uniform
#pragma unroll
          for (int u = 0; u < CW; ++u) acc[u] = mfma16(ga[s], tb[s][u], acc[u]);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ei = ib * 16 + 4 * h + v;
        if (ei < K && cok) {
          float o[CW];
#pragma unroll
          for (int u = 0; u < CW; ++u) o[u] = fmaf(gd[v], t0v[u], acc[u][v]);
          store_cols<CW>(dTb + (int64_t)(ei + 1) * d + col, o);
        }
      }
    }
  }
}

static int check_interact(const void* a, const void* b, int B, int F, int d) {
  if (!a || !b) return DLRM_ERR_NULL;
  if (B < 1 || F < 1 || F > DLRM_MAX_INTERACT_F || d < 4 || (d & 3)) return DLRM_ERR_BAD_SHAPE;
  if ((int64_t)B * F * d > ((int64_t)1 << 40)) return DLRM_ERR_BAD_SHAPE;
  return DLRM_OK;
}

// floats of LDS per wavefront: the P pair values of one sample
static int pair_stride(int F) {
  const int P = F * (F - 1) / 2;
  return P < 4 ? 4 : ((P + 3) & ~3);
}

// Forward of three and more row blocks: a wavefront per sample / W of them, us.  Small batches, whose SIMDs have one wavefront or
// none, 101 rows of 32 columns, batch 32 / 512 / 1024: 13.3 / 14.9 / 17.2 and 5.5 / 8.2 / 13.5.  From 102 rows on the pairs of four samples
// take more than half of a compute unit's 160 KB of LDS, which leaves it one workgroup of the other kernel: 102 rows of 16, batch 4096
// 45.1 / 32.4, 113 of 8, 2048 / 16384 24.9 / 19.6, 178.1 / 145.7, 113 of 32, 16384 247 / 167; 101 of 8, 2048 17.0 / 18.3.  Large batches
// where staging pays, 16384: 65 rows of 128 columns 173.5 / 151.5, 66 of 64 124 / 119, 97 of 32 143.7 / 136.7.  Where the other lines
// lie: 81 rows of 8 columns, batch 1024 / 2048 8.7 / 7.4, 10.9 / 12.0; 49 rows of 8, 512 / 1024 4.8 / 4.4, 4.8 / 5.1; 66 of 32, 4096 /
// 16384 25.1 / 22.8, 81.5 / 89.0; 34 of 32, 1024 / 4096 4.9 / 4.7, 10.0 / 11.5, of 64, 2048 / 16384 9.6 / 8.7, 49.3 / 49.8; 50 of 64, 2048 / 8192
// 15.1 / 16.1, 46.9 / 45.5, of 128, 2048 / 4096 23.5 / 24.7, 43.9 / 40.1; 90 of 32, 1100 / 2048 / 4096 16.2 / 12.5, 17.9 / 19.5,
// 34.9 / 33.5 (2048 wavefronts are two a SIMD, all that fit of the other kernel).  Three row blocks whose last stage is not full
// lose between 2048 and 3072 samples, 4096 below 96 columns, where the other kernel's last wavefronts, one for every SIMD, are most
// of 1024: 47 rows of 76 columns, 2242 / 2767 / 3470 / 5069 14.1 / 13.6, 15.2 / 16.7, 18.9 / 19.6, 27.9 / 25.3 (2900 batches: +2 to +9 %
// in what is left out, -3 and more beside it).  One chunk of 16 columns in the last stage loses longer: 36 rows of 80, 4888
// 20.1 / 22.1, 43 of 144, 2928 21.8 / 23.4.
static bool split_fwd(int F, int nb, int B, int d) {
  if (B <= 512 || kIntWaves * pair_stride(F) * 4 > 80 * 1024) return true;
  if (d < 32) return nb >= 5 && B <= 1024;
  if (nb >= 6 || B <= 1024) return true;
  if (nb == 5) return d >= 64 || B <= 4096;
  if (nb == 4) return d >= 64 && B >= (d > 64 ? 4096 : 8192);
  if (d < 64) return false;
  if (d % kSplitCols == 0 || d > 144 || (B - 1) % 1024 < 384) return true;
  return B <= 2048 || B > (d % kSplitCols == 16 ? (d < 96 ? 7168 : 4096) : d < 96 ? 4096 : 3072);
}
constexpr int kTiledPerLaunch = 1 << 23;   // samples: a launch holds fewer than 2^32 threads
template <int NB>
static int launch_fwd_split(const float* T, float* R, int B, int F, int d, hipStream_t st) {
  constexpr int W = NB > 4 ? 4 : 2;
  const int words = (16 * NB + 1) * split_stride(d), pairs = pair_stride(F);
  const size_t lds = (size_t)(words > pairs ? words : pairs) * 4;   // <= 35 KB
  const int64_t row = (int64_t)F * d, res = (int64_t)d + F * (F - 1) / 2;
  for (int64_t b0 = 0; b0 < B; b0 += kTiledPerLaunch) {
    const int n = (int)(B - b0 < kTiledPerLaunch ? B - b0 : kTiledPerLaunch);
    if (NB == 8 && d <= kSplitCols)
      hipLaunchKernelGGL((interact_fwd_split_kernel<NB, W, NB != 8>), dim3(n), dim3(W * DLRM_WAVE), lds, st,
                         T + b0 * row, R + b0 * res, F, d);
    else
      hipLaunchKernelGGL((interact_fwd_split_kernel<NB, W, true>), dim3(n), dim3(W * DLRM_WAVE), lds, st,
                         T + b0 * row, R + b0 * res, F, d);
    DLRM_CHECK_LAUNCH();
  }
  return DLRM_OK;
}

template <int NB>
static int launch_fwd(const float* T, float* R, int B, int F, int d, hipStream_t st) {
  static_assert(NB <= 7, "eight row blocks always take the split kernel");
  if constexpr (NB > 2) {
    if (split_fwd(F, NB, B, d)) return launch_fwd_split<NB>(T, R, B, F, d, st);
  }
  const int pstride = pair_stride(F);
  const size_t lds = (size_t)kIntWaves * pstride * 4;
  if (lds > 64 * 1024) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(interact_fwd_kernel<NB>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return DLRM_ERR_HIP;
  }
  hipLaunchKernelGGL((interact_fwd_kernel<NB>), dim3(div_up(B, kIntWaves)), dim3(kIntThreads), lds, st, T, R,
                     B, F, d, pstride);
  DLRM_CHECK_LAUNCH();
  return DLRM_OK;
}

constexpr int kSplitBelow = 1024;   // samples: one wavefront for each of the machine's SIMDs
// Five row blocks, where laying G out as tiles is a larger part of the work the fewer the columns: 73 rows of 16 columns,
// batch 4096 / 6000 / 16384 / 32768: 42.7 / 56.1 / 137 / 263 us with a wavefront per sample, 44.4 / 63.2 / 167 / 328 us
// with tiles; of 64 columns: 79.0 / 106 / 263 / 501 and 72.3 / 107 / 281 / 551 us; of 128 columns, 4096 / 12000 / 16384:
// 148 / 377 / 496 and 133 / 371 / 502 us.  From six blocks on tiles are level (90 rows of 4 to 16 columns: 241 and 245 us
// at batch 16384) or ahead everywhere.
constexpr int kSplitBelow5 = 4096, kSplitBelow5Wide = 12288;
// f(columns per lane and round): 4 (64-column groups) while the operand registers allow three wavefronts per SIMD (up to 4 row
// blocks: 144 registers; measured on 65 rows of 128 columns, batch 16384: 0.348 ms with 2 columns, 0.317 ms with 4), else 2 -- a
// lane then owns CW consecutive columns of 4 rows.  Narrow rows: 1 or 2 columns, so that a row's columns occupy all 16 lanes; with 4
// (five blocks and more 2) most of the instructions multiplied columns past d.  27 rows of 16 columns, batch 2048 / 16384
// 7.8 / 6.0, 36.7 / 21.1 us; 65 rows of 16, 1024 / 16384 15.8 / 8.1, 150.6 / 73.7; of 32 16.4 / 10.4, 156.0 / 103.7; 101 rows of 16
// 24.4 / 15.3, 288 / 178; 9 rows of 16, 16384 14.4 / 11.6.
template <int NB, typename F>
static void for_columns(int d, F f) {
  if (d <= 16) return f(std::integral_constant<int, 1>());
  if (d <= 32 || NB > 4) return f(std::integral_constant<int, 2>());
  if constexpr (NB <= 4) f(std::integral_constant<int, 4>());
}

template <int NB>
static int launch_bwd_tiled(const float* T, const float* dR, float* dT, int B, int F, int d, hipStream_t st) {
  constexpr int WPS = NB >= 4 ? 4 : NB;
  constexpr size_t lds = (size_t)g_words(NB) * 4;
  static_assert(lds <= 64 * 1024, "no more LDS than a launch gets without asking");
  const int64_t row = (int64_t)F * d, grad = (int64_t)d + F * (F - 1) / 2;
  for (int64_t b0 = 0; b0 < B; b0 += kTiledPerLaunch) {
    const int n = (int)(B - b0 < kTiledPerLaunch ? B - b0 : kTiledPerLaunch);
    for_columns<NB>(d, [&](auto cw) {
      hipLaunchKernelGGL((interact_bwd_tiled_kernel<NB, WPS, decltype(cw)::value>), dim3(n), dim3(WPS * DLRM_WAVE), lds, st,
                         T + b0 * row, dR + b0 * grad, dT + b0 * row, F, d);
    });
    DLRM_CHECK_LAUNCH();
  }
  return DLRM_OK;
}
template <int NB>
static int launch_bwd(const float* T, const float* dR, float* dT, int B, int F, int d, hipStream_t st) {
  static_assert(NB <= 5, "more row blocks always take the tiled kernel");
  if constexpr (NB > 1) {
    const int below = NB < 5 ? kSplitBelow : d > 64 ? kSplitBelow5Wide : kSplitBelow5;
    if (B <= below) return launch_bwd_tiled<NB>(T, dR, dT, B, F, d, st);
  }
  const int gstride = pair_stride(F);
  const size_t lds = (size_t)kIntWaves * gstride * 4;   // <= 52 KB
  for_columns<NB>(d, [&](auto cw) {
    hipLaunchKernelGGL((interact_bwd_kernel<NB, decltype(cw)::value>), dim3(div_up(B, kIntWaves)), dim3(kIntThreads), lds, st, T,
                       dR, dT, B, F, d, gstride);
  });
  DLRM_CHECK_LAUNCH();
  return DLRM_OK;
}

}  // namespace dlrm

using namespace dlrm;

extern "C" int32_t dlrm_interact_dot_fwd(const float* T, int32_t B, int32_t F, int32_t d, float* R,
                                         void* stream) {
  int st = check_interact(T, R, B, F, d);
  if (st != DLRM_OK) return st;
  if (reinterpret_cast<uintptr_t>(T) & 15) return DLRM_ERR_BAD_SHAPE;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  switch (F <= 17 ? 1 : (F + 14) / 16) {  // blocks of 16 embedding rows (all rows but the dense one)
    case 1: return launch_fwd<1>(T, R, B, F, d, hs);
    case 2: return launch_fwd<2>(T, R, B, F, d, hs);
    case 3: return launch_fwd<3>(T, R, B, F, d, hs);
    case 4: return launch_fwd<4>(T, R, B, F, d, hs);
    case 5: return launch_fwd<5>(T, R, B, F, d, hs);
    case 6: return launch_fwd<6>(T, R, B, F, d, hs);
    case 7: return launch_fwd<7>(T, R, B, F, d, hs);
    case 8: return launch_fwd_split<8>(T, R, B, F, d, hs);
  }
  return DLRM_ERR_BAD_SHAPE;
}

extern "C" int32_t dlrm_interact_dot_bwd(const float* T, const float* dR, int32_t B, int32_t F,
                                         int32_t d, float* dT, void* stream) {
  int st = check_interact(T, dR, B, F, d);
  if (st != DLRM_OK) return st;
  if (!dT) return DLRM_ERR_NULL;
  if ((reinterpret_cast<uintptr_t>(T) & 15) || (reinterpret_cast<uintptr_t>(dT) & 15))
    return DLRM_ERR_BAD_SHAPE;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  switch (F <= 17 ? 1 : (F + 14) / 16) {
    case 1: return launch_bwd<1>(T, dR, dT, B, F, d, hs);
    case 2: return launch_bwd<2>(T, dR, dT, B, F, d, hs);
    case 3: return launch_bwd<3>(T, dR, dT, B, F, d, hs);
    case 4: return launch_bwd<4>(T, dR, dT, B, F, d, hs);
    case 5: return launch_bwd<5>(T, dR, dT, B, F, d, hs);
    case 6: return launch_bwd_tiled<6>(T, dR, dT, B, F, d, hs);
    case 7: return launch_bwd_tiled<7>(T, dR, dT, B, F, d, hs);
    case 8: return launch_bwd_tiled<8>(T, dR, dT, B, F, d, hs);
  }
  return DLRM_ERR_BAD_SHAPE;
}
