// GEMMs of few tiles (bf16, k-contiguous operands): 64 x 64 tiles, operands by DMA into a ring in LDS (PipeLoop)
//   C[b][m][n] = epilogue( sum_k A[b][m][k] * B[b][n][k] ),  K a multiple of 64
//
// What bounds gemm_kernel where its 128 x 128 tiles are few (a short protein, N = 128 or 256) is the length of a workgroup's life: each
// k-step waits for its loads, stores them to LDS and passes two barriers, and nothing else on the CU fills the gaps; four to fourteen
// such steps with half of the CUs idle.  Here a step passes one barrier and finds its operands there, and four times the tiles
// fill the chip.  Per launch (us, gemm_kernel -> this): 10080 x 256, K 1024 22.7 -> 14.6, K 256 12.0 -> 8.6; 9408 x 128, K 1024 21.8 -> 11.7, K 512
// 14.7 -> 8.6, K 128 9.5 -> 6.8; 3000 x 256, K 1024 21.4 -> 9.8.  Branches one after the other, s 128, r 97 forward 378 -> 352, s 90, r 112 392 -> 358, step
// 1300 -> 1236; side by side the step 909 -> 879.
#pragma once
#include "pe_gemm.h"

constexpr int PIPE_TILE = 64;
// four waves 2 x 2, the vector epilogues of gemm_kernel
template <class Epi, int F, int S>
__global__ __launch_bounds__(256) void gemm_pipe_kernel(Operand A, Operand B, GemmShape sh, Epi epi) {
  constexpr int BM = PIPE_TILE, BN = PIPE_TILE;
  typedef PipeLoop<BM, BN, 2, S> L;
  constexpr int WS = L::TN + 4, LPR = L::TN / 8, RPI = 64 / LPR, IT = 32 / RPI;      // staging row, lanes per row, rows per step, steps
  constexpr int STG = 4 * 32 * WS * 2;      // elements
  __shared__ __attribute__((aligned(16))) bf16 lds[L::LDS > STG ? L::LDS : STG];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, g = lane >> 5;
  const int wm = (wave >> 1) * L::TM, wn = (wave & 1) * L::TN;
  // all n-tiles of a (batch, m-tile) unit on one XCD (workgroup w runs on XCD w % 8)
  const int NTm = (sh.M + BM - 1) / BM, NTn = (sh.N + BN - 1) / BN;
  const int unit = (blockIdx.x & 7) + 8 * ((blockIdx.x >> 3) / NTn);
  if (unit >= NTm * sh.batch) return;
  const int b = unit / NTm, m0 = (unit % NTm) * BM, n0 = ((blockIdx.x >> 3) % NTn) * BN;
  f32x16 acc[L::NI][L::NJ];
  L::run(acc, lds, A, (const bf16*)A.ptr + (long long)b * A.batch_stride, m0, sh.M, B, (const bf16*)B.ptr + (long long)b * B.batch_stride, n0, sh.N, sh.K);
  float* stage = reinterpret_cast<float*>(lds) + wave * 32 * WS;
  const int c8 = (lane % LPR) * 8, n = n0 + wn + c8;
  typename Epi::ColV cv;
  if (n < sh.N) epi.template colv<F>(n, cv);
#pragma unroll
  for (int i = 0; i < L::NI; i++) {
    typename Epi::Pre8 pre[IT];
#pragma unroll
    for (int it = 0; it < IT; it++) {
      const int m = m0 + wm + i * 32 + lane / LPR + it * RPI;
      if (m < sh.M && n < sh.N) epi.template pre8<F>(b, m, n, cv, pre[it]);
    }
#pragma unroll
    for (int j = 0; j < L::NJ; j++)
#pragma unroll
      for (int a = 0; a < 16; a++) stage[acc_row(g, a) * WS + j * 32 + l32] = acc[i][j][a];
    RowsPiece::phase();
#pragma unroll
    for (int it = 0; it < IT; it++) {
      const int row = lane / LPR + it * RPI, m = m0 + wm + i * 32 + row;
      if (m < sh.M && n < sh.N) {
        float vals[8];
        const f32x4 lo = *reinterpret_cast<const f32x4*>(stage + row * WS + c8), hi = *reinterpret_cast<const f32x4*>(stage + row * WS + c8 + 4);
#pragma unroll
        for (int e = 0; e < 4; e++) { vals[e] = lo[e]; vals[4 + e] = hi[e]; }
        epi.template apply8<F>(b, m, n, cv, vals, pre[it]);
      }
    }
    RowsPiece::phase();
  }
}

// A ring of three stages (48 KB, three workgroups per CU) where the tiles are at most two rounds of the CUs, of two (32 KB, five per CU) above:
// 9408 x 128, K 512 (294 tiles) 9.5 us with two, 8.6 with three; 10080 x 256, K 1024 (632) 14.6 and 16.0.
template <int F, class Epi>
static inline void launch_pipe_f(hipStream_t st, const Operand& A, const Operand& B, const GemmShape& sh, const Epi& epi) {
  const long long units = (long long)((sh.M + PIPE_TILE - 1) / PIPE_TILE) * sh.batch, ntn = (sh.N + PIPE_TILE - 1) / PIPE_TILE;
  const dim3 grid((unsigned)(8 * ((units + 7) / 8) * ntn)), block(256);
  if (units * ntn <= 512) hipLaunchKernelGGL((gemm_pipe_kernel<Epi, F, 3>), grid, block, 0, st, A, B, sh, epi);
  else hipLaunchKernelGGL((gemm_pipe_kernel<Epi, F, 2>), grid, block, 0, st, A, B, sh, epi);
  g_gemm_last_features = F;
}
static inline long long pipe_tiles(const GemmShape& sh) {
  return (long long)((sh.M + PIPE_TILE - 1) / PIPE_TILE) * ((sh.N + PIPE_TILE - 1) / PIPE_TILE) * sh.batch;
}
// Up to four rounds of tiles: with 2048 of them the two-stream step at s 128, r 256 goes from 2294 to 2331 us (64 x 64 tiles take in twice
// the operand bytes of 128 x 128 ones), with 1024 it is unchanged, and forward passes of short proteins lose nothing (352 and 352).  128 x 128 tiles
// on the same loop were 20 % faster alone from 500 tiles on (32768 x 256, K 1024 31.0 -> 24.0) and left every call as it was.
template <class Epi>
static inline bool launch_gemm_pipe(hipStream_t st, const Operand& A, const Operand& B, const GemmShape& sh, const Epi& epi) {
  if constexpr (Epi::HAS_COLSUM || Epi::TM_GATE) {
    return false;
  } else {
    if (sh.k_chunk > 0 || sh.n_rows != sh.N || pipe_tiles(sh) > 1024) return false;
    if (sh.N <= 128 && sh.M >= 128 * 256 && sh.batch == 1) return false;      // gemm64_kernel keeps the tall, narrow outputs (64 columns from 32768 rows; 36096 x 64, K 256: 11.6 us there, 9.6 here)
    if (!pipe_operand_ok(A, sh.M, sh.K) || !pipe_operand_ok(B, sh.N, sh.K)) return false;
    if constexpr (!std::is_same<Epi, EpiGeneric<bf16>>::value) {
      launch_pipe_f<0>(st, A, B, sh, epi);
      return true;
    } else {
      const int f = epi.features();
#define PE_PIPE_SPEC(S) if ((f & ~(S)) == 0) { launch_pipe_f<(S)>(st, A, B, sh, epi); return true; }
      PE_PIPE_SPEC(0)
      PE_PIPE_SPEC(EF_BIASN | EF_RES)
      PE_PIPE_SPEC(EF_BIASN | EF_ACT)
      PE_PIPE_SPEC(EF_RELUMASK)
      PE_PIPE_SPEC(EF_OM2 | EF_ON2 | EF_BIASN)
      PE_PIPE_SPEC(EF_ACC | EF_BIASM)
      PE_PIPE_SPEC(EF_BIASN | EF_ROWSCALE | EF_ON2)
      PE_PIPE_SPEC(EF_BIASN | EF_AUX | EF_MUL | EF_RES)
      PE_PIPE_SPEC(EF_OM2 | EF_ON2 | EF_ROWSCALE)
#undef PE_PIPE_SPEC
      return false;
    }
  }
}
