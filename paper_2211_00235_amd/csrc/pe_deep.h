// GEMM for large outputs with a long contraction (bf16): the three contractions of the outer product mean with many
// sequences, C[m][n] = scale2d( sum_k A[m][k] * B[n][k] ), operands k-contiguous or x-contiguous.
//
// A wave of gemm_kernel, which owns 64 x 64 of a 128 x 128 tile, reads 4 KB of fragments per four MFMAs: 128 cycles of LDS against
// 128 cycles of MFMA per 16 k of a workgroup, with the tile's stores still to come.
// Here the tile is 256 x 256 and each of eight waves owns 128 x 64 of it: 6 KB per eight MFMAs.  One workgroup per CU, two
// buffers of 64 KB: a k-step of 64 costs one barrier.  A tile is requested a whole step (64 MFMAs of each SIMD) before it is
// stored to the other buffer, and the fragments of each 16 k are requested ahead of the products of the 16 k before them.
// Counters: matrix unit busy 0.51 to 0.55 of the time at K = 5120 and 12288, LDS 0.33 to 0.35, 1.8 waves per SIMD: two waves per SIMD do not hide
// the barrier of a step; 0.25 and 0.23 at K = 512, where the epilogue, which nothing overlaps, weighs more.
// Products are summed in gemm_kernel's order: results are bit-identical to it.
#pragma once
#include "pe_gemm.h"

struct DeepCfg {
  static constexpr int BM = 256, BK = 64, TILE = BM * BK;
  // element offset in the tile of a k-contiguous operand ([row][64 k], 16-byte chunk c): 8 consecutive rows at a chunk fall on
  // all 128 bytes, 16 on all 256
  static PE_DEV int koff(int row, int c) { return row * BK + ((c ^ (row & 7) ^ ((row >> 3) & 1)) << 3); }
  // x-contiguous operand ([k][256 x], memory order): the 64-byte unit of a row XOR-ed so that the eight rows of k that a
  // transposing read touches (xfrag) fall on distinct units
  static PE_DEV int xoff(int k, int x) { return k * BM + ((((x >> 5) ^ ((k & 3) | (((k >> 3) & 1) << 2))) << 5) | (x & 31)); }
  static PE_DEV bf16x8 xfrag(const bf16* tile, int k0, int r0, int l32, int g) {
    const bf16* p = tile + xoff(k0 + 8 * g + ((l32 & 15) >> 2), r0 + (l32 & 16) + 4 * (l32 & 3));
    const bf16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 4 * BM);    // k + 4: the same unit
    bf16x8 f;
#pragma unroll
    for (int e = 0; e < 4; e++) { f[e] = lo[e]; f[4 + e] = hi[e]; }
    return f;
  }
};

// one operand's part of the staging: a thread moves four 16-byte vectors of a tile
// (a uniform base and 32-bit byte offsets: with 64-bit addresses per row the kernel spills)
template <bool KC> struct DeepTile {
  const char* base;
  unsigned ro[KC ? 4 : 1];
  unsigned ld;
  int K, c;
  // rows beyond the operand's extent X repeat the last one (their products are not stored)
  PE_DEV void init(const Operand& op, int x0, int X, int K_, int tid) {
    base = (const char*)op.ptr;
    K = K_;
    if constexpr (KC) {
      c = (tid & 7) * 8;
      ld = (unsigned)op.x_stride * 2;
#pragma unroll
      for (int i = 0; i < 4; i++) ro[i] = (unsigned)min(x0 + (tid >> 3) + 64 * i, X - 1) * ld;
    } else {
      c = tid >> 5;
      ld = (unsigned)op.k_stride * 2;
      ro[0] = (unsigned)min(x0 + (tid & 31) * 8, X - 8) * 2;
    }
  }
  // k beyond the contraction: an address inside the operand, and zeros
  PE_DEV void load(bf16x8 (&v)[4], int k0) const {
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if constexpr (KC) v[i] = *reinterpret_cast<const bf16x8*>(base + (ro[i] + (unsigned)min(k0 + c, K - 8) * 2));
      else v[i] = *reinterpret_cast<const bf16x8*>(base + (ro[0] + (unsigned)min(k0 + c + 16 * i, K - 1) * ld));
    }
  }
  PE_DEV void store(bf16x8 (&v)[4], bf16* tile, int k0, int tid) const {
    bf16x8 z;
#pragma unroll
    for (int e = 0; e < 8; e++) z[e] = (bf16)0.0f;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if constexpr (KC) *reinterpret_cast<bf16x8*>(tile + DeepCfg::koff((tid >> 3) + 64 * i, tid & 7)) = k0 + c < K ? v[i] : z;
      else *reinterpret_cast<bf16x8*>(tile + DeepCfg::xoff(c + 16 * i, (tid & 31) * 8)) = k0 + c + 16 * i < K ? v[i] : z;
    }
  }
};

template <bool A_KC, bool B_KC, int F>
__global__ __launch_bounds__(512, 2) void gemm_deep_kernel(Operand A, Operand B, GemmShape sh, EpiGeneric<bf16> epi) {
  typedef DeepCfg C;
  __shared__ __attribute__((aligned(16))) bf16 lds_all[4 * C::TILE];      // 128 KB: buffer 0 (A, B), buffer 1 (A, B)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5;
  const int wm = (wave >> 2) * 128, wn = (wave & 3) * 64;
  // an XCD (workgroup w runs on XCD w % 8) owns a run of tiles in an order that goes through four m-tiles before the next n-tile:
  // its 32 workgroups share 4 panels of A and 8 of B
  const int NTm = (sh.M + C::BM - 1) / C::BM, NTn = (sh.N + C::BM - 1) / C::BM, tiles = NTm * NTn;
  const int per = (tiles + 7) >> 3, id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || id >= tiles) return;
  const int band = id / (4 * NTn), in = id - band * 4 * NTn, bh = min(4, NTm - band * 4);
  const int m0 = (band * 4 + in % bh) * C::BM, n0 = (in / bh) * C::BM;

  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.0f;
  DeepTile<A_KC> ta;
  DeepTile<B_KC> tb;
  ta.init(A, m0, sh.M, sh.K, tid);
  tb.init(B, n0, sh.N, sh.K, tid);
  bf16x8 ra[4], rb[4], af[2][4], bf[2][2];
  auto frags = [&](const bf16* la, int kk, bf16x8 (&fa)[4], bf16x8 (&fb)[2]) {
    const bf16* lb = la + C::TILE;
#pragma unroll
    for (int j = 0; j < 2; j++) {
      if constexpr (B_KC) fb[j] = *reinterpret_cast<const bf16x8*>(lb + C::koff(wn + j * 32 + l32, 2 * kk + g));
      else fb[j] = C::xfrag(lb, kk * 16, wn + j * 32, l32, g);
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if constexpr (A_KC) fa[i] = *reinterpret_cast<const bf16x8*>(la + C::koff(wm + i * 32 + l32, 2 * kk + g));
      else fa[i] = C::xfrag(la, kk * 16, wm + i * 32, l32, g);
    }
  };
  ta.load(ra, 0);
  tb.load(rb, 0);
  ta.store(ra, lds_all, 0, tid);
  tb.store(rb, lds_all + C::TILE, 0, tid);
  ta.load(ra, C::BK);
  tb.load(rb, C::BK);
  __syncthreads();
  frags(lds_all, 0, af[0], bf[0]);
  bf16* cur = lds_all;
  bf16* nxt = lds_all + 2 * C::TILE;
  for (int k0 = 0; k0 < sh.K; k0 += C::BK) {
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
      // The fragments of the next 16 k are requested ahead of this quarter's products.  The last quarter's come from the next
      // tile: every wave has stored its part of that tile and read its last fragments of this one before the barrier.
      if (kk < 3) frags(cur, kk + 1, af[(kk + 1) & 1], bf[(kk + 1) & 1]);
      else {
        __syncthreads();
        frags(nxt, 0, af[0], bf[0]);
      }
      if (kk == 1) {      // beyond the contraction: zeros that no product reads
        ta.store(ra, nxt, k0 + C::BK, tid);
        tb.store(rb, nxt + C::TILE, k0 + C::BK, tid);
        ta.load(ra, k0 + 2 * C::BK);
        tb.load(rb, k0 + 2 * C::BK);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk & 1][i], bf[kk & 1][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    bf16* t = cur; cur = nxt; nxt = t;
  }
  __syncthreads();      // all waves are done with the operand tiles
  constexpr int WS = 68;
  float* stage = reinterpret_cast<float*>(lds_all) + wave * 32 * WS;      // 8.5 KB per wave
  const int c8 = (lane & 7) * 8, n = n0 + wn + c8;
  typename EpiGeneric<bf16>::ColV cv;
  if (n < sh.N) epi.template colv<F>(n, cv);
#pragma unroll
  for (int i = 0; i < 4; i++) {
    typename EpiGeneric<bf16>::Pre8 pre[4];
#pragma unroll
    for (int it = 0; it < 4; it++) {
      const int m = m0 + wm + i * 32 + (lane >> 3) + it * 8;
      if (m < sh.M && n < sh.N) epi.template pre8<F>(0, m, n, cv, pre[it]);
    }
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int a = 0; a < 16; a++) stage[acc_row(g, a) * WS + j * 32 + l32] = acc[i][j][a];
    RowsPiece::phase();
#pragma unroll
    for (int it = 0; it < 4; it++) {
      const int row = (lane >> 3) + it * 8, m = m0 + wm + i * 32 + row;
      if (m < sh.M && n < sh.N) {
        float vals[8];
        const f32x4 lo = *reinterpret_cast<const f32x4*>(stage + row * WS + c8), hi = *reinterpret_cast<const f32x4*>(stage + row * WS + c8 + 4);
#pragma unroll
        for (int e = 0; e < 4; e++) { vals[e] = lo[e]; vals[4 + e] = hi[e]; }
        epi.template apply8<F>(0, m, n, cv, vals, pre[it]);
      }
    }
    RowsPiece::phase();
  }
}

// Measured in the block on one stream, gemm_kernel -> this one (us; tiles of 256 x 256, share of the 256 CUs' rounds that they fill):
// both x-contiguous: 8192 x 8192, K 128 59 -> 61.5, K 256 79 -> 74, K 512 125 -> 104, K 1024 215 -> 154 (890 TFLOP/s), K 2048
// 405 -> 267; 12288 x 12288, K 170 138 -> 141, K 512 264 -> 214, K 5120 (beside the other branch) 2130 -> 1350 (1140); 3680 x 3680, K 3501
// (225 tiles, 0.88) 191 -> 109; 5120 x 5120, K 1024 (400 tiles, 0.78) 102 -> 75.  k-contiguous A: 2048 x 8192, K 8192 (256 tiles) 352 ->
// 256 and (B x-contiguous) 404 -> 243; 1024 x 9600, K 9600 (152 tiles, 0.59) 273 -> 257 and 300 -> 241; 1024 x 8192 (128 tiles, 0.5) 183 ->
// 214 and 204 -> 203; 512 x 12288 (96 tiles) 262 -> 322 and 293 -> 311.
// The share counts outputs, not tiles: in a tile wider than the output most products are of repeated rows (N 64, K 256, the input
// cotangent of a transition over 64 channels, gemm64_kernel -> this one: M 44000 10.5 -> 17.2, 262144 33 -> 60, 1966080 232 -> 432), so an
// output narrower than a tile is never taken.
// Beside another branch's kernels the same line holds (whole calls without -> with this kernel there: s 512, r 384 forward 2416 ->
// 2377, step 8624 -> 8542; s 400, r 256 forward 1172 -> 1155; extra-MSA forward at s 1024, r 256 1065 -> 1021).
static inline bool deep_fits(const Operand& A, bool a_kc, const Operand& B, bool b_kc, const GemmShape& sh) {
  if (sh.batch != 1 || sh.k_chunk > 0 || sh.n_rows != sh.N) return false;
  if (A.x_in < (1 << 30) || A.k_in < (1 << 30) || B.x_in < (1 << 30) || B.k_in < (1 << 30)) return false;
  if ((long long)sh.M * A.x_stride + (long long)sh.K * A.k_stride >= (1LL << 30) || (long long)sh.N * B.x_stride + (long long)sh.K * B.k_stride >= (1LL << 30))
    return false;      // byte offsets of 32 bits
  if ((a_kc || b_kc) && sh.K % 8) return false;
  if ((!a_kc && sh.M % 8) || (!b_kc && sh.N % 8)) return false;
  if (sh.K < 256 || sh.M < DeepCfg::BM || sh.N < DeepCfg::BM) return false;
  const long long tiles = (long long)((sh.M + 255) / 256) * ((sh.N + 255) / 256), rounds = (tiles + 255) / 256;
  return tiles < (1 << 20) && (long long)sh.M * sh.N * 20 >= rounds * 256 * 11 * (DeepCfg::BM * DeepCfg::BM);
}
template <class Epi>
static inline bool launch_gemm_deep(hipStream_t st, const Operand& A, bool a_kc, const Operand& B, bool b_kc, const GemmShape& sh, const Epi& epi) {
  if constexpr (!std::is_same<Epi, EpiGeneric<bf16>>::value) {
    return false;
  } else {
    constexpr int F = EF_SCALE2D;
    if ((epi.features() & ~F) || !deep_fits(A, a_kc, B, b_kc, sh) || (!a_kc && b_kc)) return false;
    const int tiles = ((sh.M + 255) / 256) * ((sh.N + 255) / 256);
    const dim3 grid((unsigned)((tiles + 7) / 8 * 8)), block(512);
    if (a_kc && b_kc) hipLaunchKernelGGL((gemm_deep_kernel<true, true, F>), grid, block, 0, st, A, B, sh, epi);
    else if (a_kc) hipLaunchKernelGGL((gemm_deep_kernel<true, false, F>), grid, block, 0, st, A, B, sh, epi);
    else hipLaunchKernelGGL((gemm_deep_kernel<false, false, F>), grid, block, 0, st, A, B, sh, epi);
    g_gemm_last_features = F;
    return true;
  }
}
