// Row-streaming GEMM (bf16): C[m][n] = epilogue( sum_k A[m][k] * B[n][k] ) for tall A, K = 64, 128 or 256 and a B (weights) of
// which a panel of columns fits into LDS.
//
// What bounds these GEMMs (K = channels: the projections, the first GEMM of a transition, the cotangents of hidden and gated
// tensors) is memory traffic, mostly of the output; gemm_kernel reaches 2 to 3 TB/s on them because its workgroups pass
// through load, multiply and store phases together, four k-steps each, with 16 KB of loads in flight per workgroup.  Here a
// workgroup keeps a panel of B in LDS for its whole life and its eight waves walk through 32-row blocks of A independently of
// each other, without a barrier: a wave loads its block (all of K, up to 16 KB) into registers, turns it into MFMA fragments
// through 2 KB of LDS of its own (RowsPiece; heads of 8 channels are loaded as fragments), multiplies it with the panel and
// stores; with eight waves in different phases loads, MFMAs and stores overlap.  Counters at M 196608, K 256, N 1024: 384 MiB written and 114
// fetched at 4.0 TB/s, matrix unit busy 0.32, LDS 0.35, vector unit 0.21 of the time.
//
// Products are computed transposed, D[n][m], weights as the A operand (from LDS, in fragment order: 1 KB contiguous per read)
// and rows of A as the B operand, so a row of the output is a lane (and its partner lane ^ 32): after one exchange
// of accumulator quads between the two lane halves (v_permlane32_swap) a lane holds 8 consecutive columns of its row, twice
// per 32 columns: the epilogue's arithmetic needs no LDS, its stores go through the wave's 2 KB once more.
// The products are summed over k in gemm_kernel's order: results are bit-identical to it.
#pragma once
#include "pe_gemm.h"

PE_DEV long long rows_map(int x, int in, long long outer, long long stride) {
  return in >= (1 << 30) ? (long long)x * stride : (long long)((unsigned)x / (unsigned)in) * outer + (long long)((unsigned)x % (unsigned)in) * stride;
}

template <int F> struct RowsGeneric {
  typedef EpiGeneric<bf16> E;
  static bool ok(const E& e, int N) {
    if (e.accumulate || e.alpha != 1.0f || e.scale2d || e.bias_m || e.om_used > 0 || e.out_batch) return false;
    if (e.relu_mask && !e.bits_in) return false;
    if ((e.bits_in && (e.ld_bits % 16 || ((uintptr_t)e.bits_in) % 16)) || (e.bits_out && (e.ld_bits % 4 || ((uintptr_t)e.bits_out) % 4))) return false;
    if (e.on_in < (1 << 30) && e.on_in != 8 && e.on_in % 32) return false;     // a 32-column block: four heads of 8 or part of one
    return (e.features() & ~F) == 0 && e.vec_ok(N);
  }
};

template <int F, int KS, int NP>
__global__ __launch_bounds__(512, KS <= 8 ? 4 : 2) void gemm_rows_kernel(Operand A, Operand B, GemmShape sh, EpiGeneric<bf16> epi, int npan, int groups) {
  constexpr int NC = 32 * NP;                    // columns of a panel
  constexpr int UNROLL = (F & EF_RELUMASK) ? NP / 2 : 1;      // the mask words are registers
  __shared__ __attribute__((aligned(16))) bf16 wl[NP * KS * 512];      // [column block][k step][slot][8]
  __shared__ __attribute__((aligned(16))) bf16 pl[8][1024];            // a piece per wave
  __shared__ __attribute__((aligned(16))) float bl[NC];
  __shared__ long long cl[NC / 8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5, c4 = lane & 3;
  // all panels of a group of row blocks on one XCD (workgroup w runs on XCD w % 8): its L2 serves the rows to all but the first
  const int xcd = blockIdx.x & 7, jq = blockIdx.x >> 3;
  const int panel = jq % npan, grp = (jq / npan) * 8 + xcd, n0 = panel * NC;
  const int nblk = (sh.M + 31) >> 5, step = groups * 8;
  const bf16* pa = (const bf16*)A.ptr;
  const bool k2 = A.k_in < (1 << 30), a_direct = k2 && A.k_in == 8;       // heads of 8: rows of a head are 16 bytes apart
  // a row block as loaded: pieces u (k steps 2 u, 2 u + 1) in the memory layout, or (a_direct) the fragments themselves
  bf16x8 r[KS];
  auto load_block = [&](int blk) {
    if (a_direct) {
      const bf16* ar = pa + g * A.k_outer + rows_map(min(blk * 32 + l32, sh.M - 1), A.x_in, A.x_outer, A.x_stride);
#pragma unroll
      for (int ks = 0; ks < KS; ks++) r[ks] = *reinterpret_cast<const bf16x8*>(ar + 2 * ks * A.k_outer);
    } else {
      const bf16* ar[2];
#pragma unroll
      for (int i = 0; i < 2; i++) ar[i] = pa + c4 * 8 + rows_map(min(blk * 32 + (lane >> 2) + 16 * i, sh.M - 1), A.x_in, A.x_outer, A.x_stride);
      if (k2) {
#pragma unroll
        for (int u = 0; u < KS / 2; u++)
#pragma unroll
          for (int i = 0; i < 2; i++)
            r[2 * u + i] = *reinterpret_cast<const bf16x8*>(ar[i] + (long long)((unsigned)(32 * u) / (unsigned)A.k_in) * A.k_outer + (unsigned)(32 * u) % (unsigned)A.k_in);
      } else {
#pragma unroll
        for (int u = 0; u < KS / 2; u++)
#pragma unroll
          for (int i = 0; i < 2; i++) r[2 * u + i] = *reinterpret_cast<const bf16x8*>(ar[i] + 32 * u);
      }
    }
  };
  {
    // slot of (n, g) in a fragment: the row index XOR-ed by 2 ((ks % 2) 2 + g), so that the four chunks of a 64-byte run of a row
    // of B go to distinct banks
    const bf16* pb = (const bf16*)B.ptr;
    constexpr int CHUNKS = NC * 2 * KS, PER = CHUNKS / 512;
    static_assert(CHUNKS % 512 == 0, "whole rounds of 512 threads");
#pragma unroll
    for (int i = 0; i < PER; i++) {
      const int idx = tid + i * 512;
      const int cc = idx & 3, nl = (idx >> 2) & 15, rest = idx >> 6;      // 16 rows of B x 64 bytes per wave
      const int n = (rest % (NC / 16)) * 16 + nl, c = (rest / (NC / 16)) * 4 + cc;
      *reinterpret_cast<bf16x8*>(wl + (((n >> 5) * KS + (c >> 1)) * 64 + (c & 1) * 32 + ((n & 31) ^ (cc << 1))) * 8) =
          *reinterpret_cast<const bf16x8*>(pb + (long long)(n0 + n) * B.x_stride + c * 8);
    }
    if (tid < NC) bl[tid] = ((F & EF_BIASN) && epi.bias_n && n0 + tid >= epi.bn_begin) ? epi.bias_n[n0 + tid] : 0.0f;
    if (tid < NC / 8) cl[tid] = rows_map(n0 + tid * 8, (F & EF_ON2) ? epi.on_in : (1 << 30), epi.on_outer, epi.on_stride);
  }
  __syncthreads();
  RowsPiece pc;
  pc.init(pl[wave], lane);
  const bool o_direct = (F & EF_ON2) && epi.on_in == 8;
  const int s0 = (g * 32 + (l32 ^ (g << 1))) * 8, s1 = (g * 32 + (l32 ^ ((2 + g) << 1))) * 8;   // this lane's slot at even / odd ks
  for (int blk = grp * 8 + wave; blk < nblk; blk += step) {
    load_block(blk);
    const int m = blk * 32 + l32, mc = min(m, sh.M - 1);
    const int mm[2] = {blk * 32 + (lane >> 2), blk * 32 + (lane >> 2) + 16};     // rows of the memory layout
    long long oo[2];
    bf16x8 a[KS];
#pragma unroll
    for (int u = 0; u < KS / 2; u++) {
      if (a_direct) { a[2 * u] = r[2 * u]; a[2 * u + 1] = r[2 * u + 1]; }
      else {
        const bf16x8 t[2] = {r[2 * u], r[2 * u + 1]};
        pc.to_frag(t, a[2 * u], a[2 * u + 1]);
      }
    }
#pragma unroll
    for (int i = 0; i < 2; i++) oo[i] = rows_map(mm[i], (F & EF_OM2) ? epi.om_in : (1 << 30), epi.om_outer, epi.om_stride);
    const long long od = o_direct ? rows_map(m, (F & EF_OM2) ? epi.om_in : (1 << 30), epi.om_outer, epi.om_stride) : 0;
    const float rs = ((F & EF_ROWSCALE) && epi.rowscale) ? epi.rowscale[mc] : 1.0f;
    unsigned mb[NP] = {};    // the panel's decisions of this lane's row
    if (F & EF_RELUMASK) {
#pragma unroll
      for (int q = 0; q < NP / 4; q++) {
        const uint4 t = *reinterpret_cast<const uint4*>(epi.bits_in + (long long)mc * epi.ld_bits + (n0 >> 3) + 16 * q);
        mb[4 * q] = t.x; mb[4 * q + 1] = t.y; mb[4 * q + 2] = t.z; mb[4 * q + 3] = t.w;
      }
    }
#pragma unroll UNROLL
    for (int nb = 0; nb < NP; nb += 2) {
      unsigned part[2];
      f32x16 acc[2];
#pragma unroll
      for (int p = 0; p < 2; p++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[p][e] = 0.0f;
      int wo = nb * KS * 512;
      asm volatile("" : "+v"(wo));   // or a panel of two blocks is hoisted out of the row loop into registers, and spills
      const bf16* w0 = wl + wo + s0;
      const bf16* w1 = wl + wo + s1;
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        const bf16* w = (ks & 1) ? w1 : w0;
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(w + ks * 512), a[ks], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(w + (KS + ks) * 512), a[ks], acc[1], 0, 0, 0);
      }
#pragma unroll
      for (int p = 0; p < 2; p++) {
        part[p] = 0;
        const int nl = (nb + p) * 32;
        bf16x8 o[2];
#pragma unroll
        for (int j = 0; j < 2; j++) {
          float v[8];
          rows_unpack(acc[p], j, v);
          if (F & EF_BIASN) {
            const f32x4 b0 = *reinterpret_cast<const f32x4*>(bl + nl + 16 * j + 8 * g), b1 = *reinterpret_cast<const f32x4*>(bl + nl + 16 * j + 8 * g + 4);
#pragma unroll
            for (int i = 0; i < 4; i++) { v[i] += b0[i]; v[4 + i] += b1[i]; }
          }
          if (F & EF_ACT) {
            if (epi.act == 1) {
              unsigned bb = 0;
#pragma unroll
              for (int i = 0; i < 8; i++) {
                v[i] = fmaxf(v[i], 0.0f);
                bb |= (to_f(from_f<bf16>(v[i])) > 0.0f ? 1u : 0u) << i;   // the decision of the STORED value
              }
              part[p] |= bb << (8 * (2 * j + g));
            } else if (epi.act == 2) {
#pragma unroll
              for (int i = 0; i < 8; i++) v[i] = sigmoidf_(v[i]);
            }
          }
          if (F & EF_RELUMASK) {
            const unsigned bits = mb[nb + p] >> (8 * (2 * j + g));
#pragma unroll
            for (int i = 0; i < 8; i++) v[i] = ((bits >> i) & 1u) ? v[i] : 0.0f;
          }
          if (F & EF_ROWSCALE) {
#pragma unroll
            for (int i = 0; i < 8; i++) v[i] *= rs;
          }
#pragma unroll
          for (int i = 0; i < 8; i++) o[j][i] = from_f<bf16>(v[i]);
        }
        if (o_direct) {
#pragma unroll
          for (int j = 0; j < 2; j++)
            if (m < sh.M) *reinterpret_cast<bf16x8*>(epi.out + od + cl[(nl >> 3) + 2 * j + g]) = o[j];
        } else {
          bf16x8 t[2];
          pc.to_mem(o, t[0], t[1]);
          const long long co = cl[(nl >> 3) + c4];
#pragma unroll
          for (int i = 0; i < 2; i++)
            if (mm[i] < sh.M) *reinterpret_cast<bf16x8*>(epi.out + oo[i] + co) = t[i];
        }
      }
      if ((F & EF_ACT) && epi.bits_out) {   // lane half g stores the 32 decisions of column block nb + g
        const auto r = __builtin_amdgcn_permlane32_swap(part[0], part[1], false, false);
        if (m < sh.M) *reinterpret_cast<unsigned*>(epi.bits_out + (long long)m * epi.ld_bits + ((n0 + (nb + g) * 32) >> 3)) = r[0] | r[1];
      }
    }
  }
}

// Operands the kernel takes (the epilogue is checked by the launcher).
// Beside another branch's kernels (sh.beside) the waves and the LDS it keeps are room that the other stream's workgroups would
// have filled: K >= 128 pays there only where the launch is long, so outputs of more than 2^26 elements.  Whole calls, none -> these:
// s 512, r 384 step 8868 -> 8542 us, forward 2627 -> 2377; s 400, r 200 step 3347 -> 3265; s 400, r 256 4364 -> 4207.  (From 2^25: s 256, r 256
// 3227 -> 3138, but s 128, r 256, of which every GEMM is below, 2338 -> 2390 with all of them.)  K = 64 pays beside as it does alone: extra-MSA
// step at s 1024, r 256 3379 -> 3344, s 2000, r 70 1467 -> 1449.
// Epilogues that read a tensor of the output's size gain nothing (N = K = 256 with a residual, M 196608: 63.6 -> 67.4), nor do outputs
// of 64 columns (M 262144, K 256: 39.6 -> 41.8): not taken.
static inline bool rows_operands_ok(const Operand& A, const Operand& B, const GemmShape& sh) {
  if (sh.batch != 1 || sh.k_chunk > 0 || sh.n_rows != sh.N) return false;
  if (sh.K != 64 && sh.K != 128 && sh.K != 256) return false;
  if (sh.N % 128 || B.x_in < (1 << 30) || B.k_in < (1 << 30) || B.x_stride < sh.K) return false;
  if (A.k_in < (1 << 30) && A.k_in != 8 && A.k_in % 32) return false;
  if (sh.beside && sh.K >= 128 && (long long)sh.M * sh.N <= (1LL << 26)) return false;
  return sh.K != 256 || sh.N % 256 == 0;
}
// Launches alone on the chip, gemm_kernel or gemm64_kernel -> this one (us; plain = head-major projections, act = activation, mask = decisions
// on the way in): K 256, N 1024: plain M 12800 22.6 -> 17.6, 32768 34 -> 28, 196608 232 -> 142 (4.0 TB/s), act 12800 25.0 -> 19.9, 32768 38 -> 34,
// mask 10240 18.4 -> 17.8, 32768 45 -> 31.  K 128, N 512: plain M 2304 9.5 -> 8.6, 65536 28 -> 21, act 2304 10.7 -> 10.2, 33124 23.6 -> 18.1, mask 65536
// 34 -> 24; N 1024: M 1024 10.6 -> 9.3, 65536 44 -> 32; N 128: plain M 65536 12.0 -> 10.9, 147456 18.5 -> 18.8.  K 64, N 256: plain M 24000 10.8 -> 10.2,
// 65536 17.5 -> 13.2, 1966080 310 -> 250, act 51200 18.4 -> 15.3, 262144 49 -> 45, 1966080 354 -> 361 (without decisions 355 -> 329), mask 51200
// 18.1 -> 13.8, 1966080 432 -> 312.
// At K = 256 the first block waits for a panel of 128 KB: the row blocks of all panels have to fill more than half of the 2048 wave slots.
// An activation on the way out lengthens a wave's life, and the kernel loses where the one it replaces needs a single round of workgroups
// (768 of gemm_kernel are resident at once, as many of gemm64_kernel), or where its own waves need a second round that they hardly fill:
//   K 64, panels of 256 columns, up to 768 tiles of 128 x 128: M 8192 9.9 -> 12.3, 32768 11.7 -> 14.0, 44800 13.3 -> 13.9 (whole forward passes 269.5 -> 272.0,
//     359 -> 361.5, 408.7 -> 409.0); above: 51200 18.4 -> 15.3
//   K 256, up to 768 tiles: N 1024 M 10240 18.0 -> 20.4, 12288 19.1 -> 20.4 (forward 313.5 -> 315.2, 319.0 -> 320.5); N 2048 M 5120 18.9 -> 20.1
//   K 256, 2049 to 2560 waves: N 1024 M 18432 28.4 -> 31.4 (forward 385 -> 390), 20480 29.2 -> 31.2 (398 -> 401), 21120 (2640 waves) forward 413 -> 410; N 512
//     M 34560 27.5 -> 31.7
//   N 128 on gemm64_kernel (M from 32768), up to 768 of its 64-row tiles: K 128 M 33856 10.6 -> 11.2, 40000 11.2 -> 11.7 (forward 476.9 -> 480.9, 507.0 ->
//     510.3); K 64 M 32768 8.6 -> 10.2; above: K 128 M 50176 12.5 -> 12.2
// Plain outputs and masks were neutral or better in whole calls on both sides of these lines (within 0.2 %).
static inline bool rows_pays(const GemmShape& sh, int features) {
  const bool act = features & EF_ACT;
  const int M = sh.M;
  const long long tiles = (long long)((M + 127) / 128) * (sh.N / 128);      // gemm_kernel's workgroups
  if (act && sh.K == 64 && sh.N % 256 == 0 && tiles <= 768) return false;
  if (act && sh.N == 128 && M >= 128 * 256 && M <= 768 * 64) return false;
  if (sh.K == 256) {
    const long long waves = (long long)((M + 31) / 32) * (sh.N / 256);
    if (waves < 1280 || (act && (tiles <= 768 || (waves > 2048 && waves <= 2560)))) return false;
  }
  return true;
}
// NP: panel width in 32-column blocks.  K = 256: 128 KB of LDS, one workgroup per CU; else at most 50 KB and at most 128 registers,
// two workgroups per CU (K = 128 with 256-column panels: 166 registers, one workgroup, M 147456 N 512 49 us instead of 42)
template <int F, int KS, int NP>
static inline void launch_rows_np(hipStream_t st, const Operand& A, const Operand& B, const GemmShape& sh, const EpiGeneric<bf16>& epi) {
  const int npan = sh.N / (32 * NP), per_cu = KS <= 8 ? 2 : 1;
  const long long waves8 = ((long long)(sh.M + 31) / 32 + 7) / 8;                 // workgroups that one round of all row blocks fills
  long long groups = std::max(1, 256 * per_cu / npan / 8) * 8LL;
  groups = std::min(groups, (waves8 + 7) / 8 * 8);
  hipLaunchKernelGGL((gemm_rows_kernel<F, KS, NP>), dim3((unsigned)(groups * npan)), dim3(512), 0, st, A, B, sh, epi, npan, (int)groups);
}
template <int F>
static inline bool launch_rows_f(hipStream_t st, const Operand& A, const Operand& B, const GemmShape& sh, const EpiGeneric<bf16>& epi) {
  if (!RowsGeneric<F>::ok(epi, sh.N) || !rows_pays(sh, epi.features())) return false;
  if (sh.K == 256) launch_rows_np<F, 16, 8>(st, A, B, sh, epi);
  else if (sh.K == 128) launch_rows_np<F, 8, 4>(st, A, B, sh, epi);
  else if (sh.N % 256 == 0) launch_rows_np<F, 4, 8>(st, A, B, sh, epi);
  else launch_rows_np<F, 4, 4>(st, A, B, sh, epi);
  g_gemm_last_features = F;
  return true;
}
template <class Epi>
static inline bool launch_gemm_rows(hipStream_t st, const Operand& A, const Operand& B, const GemmShape& sh, const Epi& epi) {
  if constexpr (!std::is_same<Epi, EpiGeneric<bf16>>::value) {
    return false;
  } else {
    if (!rows_operands_ok(A, B, sh)) return false;
    return launch_rows_f<0>(st, A, B, sh, epi) || launch_rows_f<EF_BIASN | EF_ACT>(st, A, B, sh, epi) ||
           launch_rows_f<EF_RELUMASK>(st, A, B, sh, epi) || launch_rows_f<EF_OM2 | EF_ON2 | EF_BIASN>(st, A, B, sh, epi) ||
           launch_rows_f<EF_OM2 | EF_ON2 | EF_ROWSCALE>(st, A, B, sh, epi);
  }
}
