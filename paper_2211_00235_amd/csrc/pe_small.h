// GEMM for small problems: C[b][m][n] = epilogue( sum_k A[b][m][k] * B[b][n][k] ) with the operands, shapes and epilogues of
// pe_gemm.h, one 32 x 32 output tile per workgroup.
//
// What bounds a small GEMM is the length of one workgroup's life, not any throughput: with the 128 x 128 kernel a launch of
// 24 workgroups and K = 32 took 8 us, most of it straight-line code that every launch fetches cold (the instruction cache
// does not outlive a launch) and barrier-separated stages that nothing else fills.  Here the operand fragments go from
// memory straight into registers (no LDS tiles, no barrier before the epilogue), all loads of four k-chunks are in flight
// at once, the waves of a workgroup split the contraction, and the epilogue is one short loop.
// A fragment is VEC consecutive k of one row per lane: k = 2 VEC chunk + VEC g + e for lane group g.  The contraction index may be
// permuted as long as both operands agree, so 32-bit operands use the same 16-byte loads as 16-bit ones: element e of the
// two vectors feeds the e-th 32x32x2 MFMA.
#pragma once
#include "pe_elem.h"
#include "pe_gemm.h"

// LayerNorm of the A rows on the way in (K = channels <= SMALL_LN_K, rows of A contiguous): every lane holds half a row.
template <typename T> struct SmallLn { const float* gamma; const float* beta; T* y; float* stats; float eps; };
template <typename T> constexpr int small_ln_k() { return 16 * Vec16<T>::N; }   // 64 (fp32) or 128 (bf16)

// GEMM value (+ prev) = cotangent dy of a LayerNorm output, N = channels <= 32: what gemm64r_kernel's MODE 2 does, on a 32-row tile
template <typename T> struct EpiLnBwd {
  static constexpr bool HAS_COLSUM = false;
  RowLn<T> ln;
  // dy may be the sum of two products (the triangle multiplication's projection and gate paths): K2 > 0 adds A2 B2^T (vector operands)
  Operand A2, B2; int K2;
  struct Row {}; struct Col {}; struct ColV {}; struct Pre8 {};
};
template <class Epi> struct is_ln_bwd { static constexpr bool value = false; };
template <typename T> struct is_ln_bwd<EpiLnBwd<T>> { static constexpr bool value = true; };

// Loads outside the operand read its first element instead and are replaced by zero: with a branch around every load the compiler
// waits for each before it issues the next.
template <typename T, bool AV> PE_DEV typename Vec16<T>::type small_load(const T* base, const Operand& op, long long ra, bool ok, int k, int kend) {
  typedef typename Vec16<T>::type V;
  constexpr int VEC = Vec16<T>::N;
  V v;
  if (AV) {
    const bool in = ok && k < kend;
    v = *reinterpret_cast<const V*>(base + (in ? ra + gemm_kaddr(op, k) : 0));
#pragma unroll
    for (int e = 0; e < VEC; e++) v[e] = in ? v[e] : from_f<T>(0.0f);
  } else {
#pragma unroll
    for (int e = 0; e < VEC; e++) {
      const bool in = ok && k + e < kend;
      const T t = base[in ? ra + gemm_kaddr(op, k + e) : 0];
      v[e] = in ? t : from_f<T>(0.0f);
    }
  }
  return v;
}
PE_DEV void small_mma(f32x16& acc, const bf16x8& a, const bf16x8& b) { Mma<bf16>::mma(acc, a, b); }
PE_DEV void small_mma(f32x16& acc, const f32x4& a, const f32x4& b) {
#pragma unroll
  for (int e = 0; e < 4; e++) Mma<float>::mma(acc, a[e], b[e]);
}
PE_DEV long long small_xaddr(const Operand& op, int x) {
  return (op.x_in >= (1 << 30)) ? (long long)x * op.x_stride
                                : (long long)((unsigned)x / (unsigned)op.x_in) * op.x_outer + (long long)((unsigned)x % (unsigned)op.x_in) * op.x_stride;
}

constexpr int SMALL_WS = 36;   // row stride of a staged 32 x 32 tile
// AV / BV: the operand's k is contiguous and 16-byte vectors of it are aligned (else element loads, coalesced over the rows where
// those are contiguous); VE: the vector epilogue applies; LN: LayerNorm of the A rows on the way in (every wave normalises the
// whole rows, which costs no latency, and multiplies its share of the chunks).  At least two waves: threads 0..127 own one
// group of 8 output columns each and fetch its epilogue operands first of all.
template <typename T, bool AV, bool BV, bool VE, class Epi, bool LN>
__global__ __launch_bounds__(512) void gemm_small_kernel(Operand A, Operand B, GemmShape sh, Epi epi, SmallLn<T> ln) {
  typedef typename Vec16<T>::type V;
  constexpr int VEC = Vec16<T>::N, KCH = 2 * VEC;
  constexpr bool LNB = is_ln_bwd<Epi>::value;
  extern __shared__ __attribute__((aligned(16))) float small_lds[];   // [waves][32][SMALL_WS]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int l32 = lane & 31, g = lane >> 5;
  const int m0 = blockIdx.x * 32, n0 = blockIdx.y * 32, b = blockIdx.z;
  int kbeg = 0, kend = sh.K;
  const T* pa = (const T*)A.ptr;
  const T* pb = (const T*)B.ptr;
  if (sh.k_chunk > 0) {
    kbeg = b * sh.k_chunk;
    kend = min(sh.K, kbeg + sh.k_chunk);
  } else {
    pa += (long long)b * A.batch_stride;
    pb += (long long)b * B.batch_stride;
  }
  const int m = m0 + l32, n = n0 + l32;
  const bool aok = m < sh.M, bok = n < sh.n_rows;
  const long long ra = small_xaddr(A, aok ? m : 0), rb = small_xaddr(B, bok ? n : 0);
  // this thread's group of the output tile
  const int erow = (tid & 127) >> 2, ec8 = (tid & 3) * 8, em = m0 + erow, en = n0 + ec8;
  const bool eok = tid < 128 && em < sh.M && en < sh.N;
  typename Epi::ColV cv;
  typename Epi::Pre8 pre;
  if constexpr (VE && !LNB) {
    if (eok) {
      epi.template colv<EF_ALL>(en, cv);
      epi.template pre8<EF_ALL>(b, em, en, cv, pre);
    }
  }
  Raw8<T> xr, gr, pr;
  float mean = 0.0f, rstd_in = 0.0f;
  if constexpr (LNB) {
    xr.zero(); gr.zero(); pr.zero();
    if (eok) {
      const long long o0 = (long long)em * sh.N + ec8;
      xr.ld(epi.ln.x + o0);
      if (epi.ln.gin) gr.ld(epi.ln.gin + o0);
      if (epi.ln.prev) pr.ld(epi.ln.prev + o0);
      mean = epi.ln.stats_in[(long long)em * 2]; rstd_in = epi.ln.stats_in[(long long)em * 2 + 1];
    }
  }
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; e++) acc[e] = 0.0f;
  float cs = 0.0f;
  const int nc = (kend - kbeg + KCH - 1) / KCH;
  if constexpr (LN) {
    constexpr int NC = small_ln_k<T>() / KCH;
    V av[NC], bv[NC / 2];
#pragma unroll
    for (int c = 0; c < NC; c++)
      if (c < nc) av[c] = small_load<T, AV>(pa, A, ra, aok, c * KCH + g * VEC, kend);
#pragma unroll
    for (int c = 0; c < NC / 2; c++)      // wave w of two multiplies the chunks 2 c + w
      if (2 * c < nc) bv[c] = small_load<T, BV>(pb, B, rb, bok, (2 * c + wave) * KCH + g * VEC, kend);
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < NC; c++)
      if (c < nc) {
#pragma unroll
        for (int e = 0; e < VEC; e++) s += to_f(av[c][e]);
      }
    const float mu = (s + __shfl_xor(s, 32, 64)) / (float)sh.K;
    float q = 0.0f;
#pragma unroll
    for (int c = 0; c < NC; c++)
      if (c * KCH + g * VEC < kend) {
#pragma unroll
        for (int e = 0; e < VEC; e++) { const float t = to_f(av[c][e]) - mu; q += t * t; }
      }
    const float rstd = rsqrtf((q + __shfl_xor(q, 32, 64)) / (float)sh.K + ln.eps);
    const bool wr = ln.y && n0 == 0 && aok;
#pragma unroll
    for (int c = 0; c < NC; c++)
      if ((c & 1) == wave && c < nc) {   // uniform: every lane takes part in the MFMA
        const int k = c * KCH + g * VEC;
        if (k < kend) {
#pragma unroll
          for (int e = 0; e < VEC; e++) av[c][e] = from_f<T>((to_f(av[c][e]) - mu) * rstd * ln.gamma[k + e] + ln.beta[k + e]);
          if (wr) *reinterpret_cast<V*>(ln.y + (long long)m * sh.K + k) = av[c];
        }
        small_mma(acc, av[c], bv[c >> 1]);
      }
    if (wr && wave == 0 && g == 0) { ln.stats[(long long)m * 2] = mu; ln.stats[(long long)m * 2 + 1] = rstd; }
  } else {
    for (int c = wave; c < nc; c += 4 * nw) {
      V av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int k = kbeg + (c + i * nw) * KCH + g * VEC;
        av[i] = small_load<T, AV>(pa, A, ra, aok, k, kend);
        bv[i] = small_load<T, BV>(pb, B, rb, bok, k, kend);
      }
#pragma unroll
      for (int i = 0; i < 4; i++) {
        small_mma(acc, av[i], bv[i]);
        if constexpr (Epi::HAS_COLSUM) {
#pragma unroll
          for (int e = 0; e < VEC; e++) cs += to_f(bv[i][e]);
        }
      }
    }
    if constexpr (LNB) {
      const T* pa2 = (const T*)epi.A2.ptr;
      const T* pb2 = (const T*)epi.B2.ptr;
      for (int k = wave * KCH + g * VEC; k - g * VEC < epi.K2; k += nw * KCH)
        small_mma(acc, small_load<T, true>(pa2, epi.A2, small_xaddr(epi.A2, aok ? m : 0), aok, k, epi.K2),
                  small_load<T, true>(pb2, epi.B2, small_xaddr(epi.B2, bok ? n : 0), bok, k, epi.K2));
    }
  }
  float* stage = small_lds + wave * 32 * SMALL_WS;
#pragma unroll
  for (int a = 0; a < 16; a++) stage[acc_row(g, a) * SMALL_WS + l32] = acc[a];
  if constexpr (Epi::HAS_COLSUM) {   // the sums over k of the B rows, beside the wave's tile
    cs += __shfl_xor(cs, 32, 64);
    if (g == 0) stage[l32 * SMALL_WS + 32] = cs;
  }
  __syncthreads();
  if (!LNB && tid >= 128) return;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; e++) v[e] = 0.0f;
  for (int w = 0; w < nw && tid < 128; w++)
#pragma unroll
    for (int e = 0; e < 8; e++) v[e] += small_lds[(w * 32 + erow) * SMALL_WS + ec8 + e];
  if constexpr (LNB) {
    // a row of at most 32 channels is four neighbouring lanes
    const RowLn<T>& L = epi.ln;
    const int Cc = sh.N;
    float dg[8], xh[8], o[8], s1 = 0.0f, s2 = 0.0f;
    pr.get(o);
    xr.get(xh);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      v[e] = eok ? to_f(from_f<T>(v[e] + o[e])) : 0.0f;   // as the separate kernels store it
      xh[e] = (xh[e] - mean) * rstd_in;
      dg[e] = v[e] * xh[e];
      const float dx = eok ? v[e] * L.gamma[ec8 + e] : 0.0f;
      s1 += dx;
      s2 += dx * xh[e];
    }
    s1 += __shfl_xor(s1, 1, 64); s1 += __shfl_xor(s1, 2, 64);
    s2 += __shfl_xor(s2, 1, 64); s2 += __shfl_xor(s2, 2, 64);
    s1 /= (float)Cc; s2 /= (float)Cc;
    if (eok) {
      gr.get(o);
#pragma unroll
      for (int e = 0; e < 8; e++) o[e] += (v[e] * L.gamma[ec8 + e] - s1 - xh[e] * s2) * rstd_in;
      store8<T>(L.gout + (long long)em * Cc + ec8, o);
    }
    // gain / offset gradients of the tile's rows: 16 lanes of a wave, then waves 0 and 1
    float* red = small_lds + nw * 32 * SMALL_WS;   // [2][64]
#pragma unroll
    for (int e = 0; e < 8; e++) {
#pragma unroll
      for (int x = 4; x < 64; x <<= 1) { dg[e] += __shfl_xor(dg[e], x, 64); v[e] += __shfl_xor(v[e], x, 64); }
    }
    if (lane < 4 && wave < 2) {
#pragma unroll
      for (int e = 0; e < 8; e++) { red[wave * 64 + ec8 + e] = dg[e]; red[wave * 64 + 32 + ec8 + e] = v[e]; }
    }
    __syncthreads();
    if (tid < 64 && l32 < Cc) L.partial[(long long)blockIdx.x * 2 * Cc + g * Cc + l32] = red[tid] + red[64 + tid];
  } else {
    if constexpr (Epi::HAS_COLSUM) {
      if (epi.want_colsum() && blockIdx.x == 0 && tid < 32 && n0 + tid < sh.N) {
        float t = 0.0f;
        for (int w = 0; w < nw; w++) t += small_lds[(w * 32 + tid) * SMALL_WS + 32];
        epi.put_colsum(b, n0 + tid, sh.N, t);
      }
    }
    if (eok) {
      if constexpr (VE) {
        epi.template apply8<EF_ALL>(b, em, en, cv, v, pre);
      } else {
        const typename Epi::Row r = epi.row(b, em);
#pragma unroll
        for (int e = 0; e < 8; e++)
          if (en + e < sh.N) epi(em, en + e, r, epi.col(en + e), v[e]);
      }
    }
  }
}

// Which GEMMs take it: those whose 32 x 32 tiles (tiles x batch) are few and whose contraction over all of them is short (every tile
// loads its own operand rows, nothing is shared through LDS).  Measured alone on the chip against the 128 x 128 kernel (us): bf16
// 1152 x 128 x 32: 3.9 / 6.4, 2048 x 256 x 1024 (512 tiles) 10.7 / 18.7, 8192 x 128 x 512 (1024) 10.7 / 12.1, 2048 x 1024 x 256 (2048) 11.5 / 9.0;
// fp32 1152 x 128 x 32: 4.9 / 7.7, 2048 x 1024 x 256 23.5 / 25.5, 8192 x 512 x 128 (4096) 26 / 18.
// x-contiguous operands are loaded element by element: fewer tiles (fp32 parameter gradients 64 x 64 x 4096 in 128 splits, 512 tiles:
// 5.2 / 6.2, 256 x 1024 x 1024 in 16, 4096 tiles: 15 / 12; bf16 64 x 64 x 4096, 256 tiles: 5.4 / 5.1).
template <typename T> static inline bool small_gemm_fits(long long M, long long N, long long K, long long batch, bool a_kc, bool b_kc) {
  const long long tiles = ((M + 31) / 32) * ((N + 31) / 32) * batch;
  const long long most = sizeof(T) == 2 ? (a_kc && b_kc ? 1024 : 256) : (a_kc && b_kc ? 2048 : 512);
  return tiles <= most && K <= 2048 && tiles * K <= (1 << 19) && batch <= 65535;
}
// waves that share a tile's contraction: about two rounds of four chunks each, at most eight
template <typename T> static inline int small_gemm_waves(long long K) {
  const long long per = sizeof(T) == 2 ? 128 : 32;
  int nw = 2;
  while (nw < 8 && K / nw > per) nw *= 2;
  return nw;
}
template <typename T> static inline bool small_vec_operand(const Operand& o, bool kc, int X, const GemmShape& sh) {
  return kc && gemm_operand_ok<T>(o, true, X, sh);
}
template <typename T, class Epi>
static inline void launch_gemm_small(hipStream_t st, const Operand& A, bool a_kc, const Operand& B, bool b_kc, const GemmShape& sh, const Epi& epi) {
  const bool av = small_vec_operand<T>(A, a_kc, sh.M, sh), bv = small_vec_operand<T>(B, b_kc, sh.n_rows, sh), ve = epi.vec_ok(sh.N);
  const int nw = small_gemm_waves<T>(sh.k_chunk > 0 ? sh.k_chunk : sh.K);
  const dim3 grid((sh.M + 31) / 32, (sh.N + 31) / 32, sh.batch), block(64 * nw);
  const unsigned lds = (unsigned)(nw * 32 * SMALL_WS * sizeof(float));
  const SmallLn<T> ln{};
#define PE_SMALL(AV, BV, VE) hipLaunchKernelGGL((gemm_small_kernel<T, AV, BV, VE, Epi, false>), grid, block, lds, st, A, B, sh, epi, ln)
  if (ve) {
    if (av && bv) PE_SMALL(true, true, true); else if (av) PE_SMALL(true, false, true);
    else if (bv) PE_SMALL(false, true, true); else PE_SMALL(false, false, true);
  } else if constexpr (Epi::ELEM) {
    if (av && bv) PE_SMALL(true, true, false); else if (av) PE_SMALL(true, false, false);
    else if (bv) PE_SMALL(false, true, false); else PE_SMALL(false, false, false);
  }
#undef PE_SMALL
}
// LayerNorm of A's rows (contiguous, K channels) + GEMM; false: not launched
template <typename T>
static inline bool launch_gemm_small_ln(hipStream_t st, const Operand& A, const Operand& B, const GemmShape& sh, const EpiGeneric<T>& epi, const SmallLn<T>& ln) {
  if (sh.batch != 1 || sh.K > small_ln_k<T>() || !small_gemm_fits<T>(sh.M, sh.N, sh.K, 1, true, true)) return false;
  if (!small_vec_operand<T>(A, true, sh.M, sh) || !small_vec_operand<T>(B, true, sh.N, sh) || !epi.vec_ok(sh.N) || ((uintptr_t)ln.y) % 16) return false;
  hipLaunchKernelGGL((gemm_small_kernel<T, true, true, true, EpiGeneric<T>, true>), dim3((sh.M + 31) / 32, (sh.N + 31) / 32), dim3(128),
                     (unsigned)(2 * 32 * SMALL_WS * sizeof(float)), st, A, B, sh, epi, ln);
  return true;
}
// GEMM (or the sum of two: A2 != nullptr) + LayerNorm backward on rows of at most 32 channels; partials: one per 32 rows.
// false: not launched
template <typename T>
static inline bool launch_gemm_small_lnb(hipStream_t st, const Operand& A, bool a_kc, const Operand& B, const GemmShape& sh, const RowLn<T>& ln,
                                         const Operand* A2 = nullptr, const Operand* B2 = nullptr, int K2 = 0) {
  auto p16 = [](const void* p) { return ((uintptr_t)p) % 16 == 0; };
  const bool av = small_vec_operand<T>(A, a_kc, sh.M, sh);
  if ((a_kc && !av) || !small_vec_operand<T>(B, true, sh.N, sh)) return false;
  if (!p16(ln.x) || !p16(ln.gout) || !p16(ln.gin) || !p16(ln.prev)) return false;
  EpiLnBwd<T> e;
  e.ln = ln; e.A2 = A; e.B2 = B; e.K2 = 0;
  if (A2) {
    GemmShape s2 = sh;
    s2.K = K2;
    if (!small_vec_operand<T>(*A2, true, sh.M, s2) || !small_vec_operand<T>(*B2, true, sh.N, s2)) return false;
    e.A2 = *A2; e.B2 = *B2; e.K2 = K2;
  }
  const int nw = small_gemm_waves<T>(sh.K);
  const dim3 grid((sh.M + 31) / 32), block(64 * nw);
  const unsigned lds = (unsigned)((nw * 32 * SMALL_WS + 128) * sizeof(float));
  if (av) hipLaunchKernelGGL((gemm_small_kernel<T, true, true, true, EpiLnBwd<T>, false>), grid, block, lds, st, A, B, sh, e, SmallLn<T>{});
  else hipLaunchKernelGGL((gemm_small_kernel<T, false, true, true, EpiLnBwd<T>, false>), grid, block, lds, st, A, B, sh, e, SmallLn<T>{});
  return true;
}
