// Gated multi-head attention with optional pair bias and key mask: forward and backward.
//
// Used four ways by the block: MSA row attention (bias from the pair representation),
// MSA column attention (no bias, strided sequence axis), triangle attention around the
// starting node and around the ending node (strided axes + transposed bias).
//
// Data layout: HEAD-MAJOR.  q, k, v and the gate pre-activation live in one tensor `qkvg` of
// 4*H planes [B*L][d]; element (which w, head h, batch b, position p, channel c) is at
//   qkvg + (w*H + h)*plane + (b*L + p)*d + c,      plane = B*L*d.
// o / og / dO / dog are H planes of the same shape.  A head's K, V, Q tile is therefore one
// contiguous run of memory (64 positions x 64 bytes at d = 32) whatever axis the attention runs
// along; the producing / consuming GEMMs reach this layout through their two-level index maps.
// (With channel-last [B*L][4*H*d] rows a head's 64-byte slice sits alone in its 128-byte line:
// measured HBM fetch of the forward kernel was 2.5x its algorithmic bytes.)
//
// Kernel design (gfx950): every wave owns 32 queries (or 32 keys in the dK/dV kernel) and
// computes TRANSPOSED score tiles S^T = K Q^T with v_mfma 32x32, so that a query is a
// lane (column) and its keys are spread over the lane's 16 accumulator elements and the
// partner lane (lane ^ 32).  Row max / row sum then need one cross-lane exchange, the
// per-query softmax state is one scalar per lane, and the probability tile can be fed
// straight back as an MFMA operand (the contraction index is permuted consistently on
// both operands; the other operand, V / K / Q / dO with channels as rows, comes from the row-major LDS
// tile by transposing reads in bf16, from a transposed LDS copy in fp32 and in the walking backward).
// Online softmax over key tiles of 32 out of staged chunks.
#pragma once
#include "pe_common.h"
#include "pe_elem.h"

struct AttnArgs {
  const void* qkvg; long long plane;    // plane = B*L*d elements
  int B, L, H, d;
  // pair bias, multiplied by log2 e, storage type, in the two layouts that bias_tile_kernel writes (nullptr: no bias):
  const void* biasQ;                 // [H][key tile][chunk][g][query][CH]: read by the query-per-lane kernels
  const void* biasK;                 // [H][query tile][chunk][g][key][CH]: read by the key-per-lane kernel
  const float* mask; long long mask_bs, mask_ks;   // key mask value at mask[b*mask_bs + j*mask_ks]
  void* o; void* og;                 // forward outputs (o ungated, og = sigmoid(g) * o); the forward kernel takes o, lse = nullptr:
  float* lse;                        // [B][H][L]              not stored (only a backward pass reads them)
  float scale;                       // 1/sqrt(d)
  // backward
  const void* dog;                   // cotangent of og
  void* dO;                          // scratch: cotangent of o (written by pre kernel)
  float* D;                          // [B][H][L] rowsum(dO * o)
  void* dqkvg;                       // same layout as qkvg
  void* dS;                          // [ceil(B/2)][H] planes in the layout of biasQ (storage type), biased attention only
};

// XCD-aware decode of the 1-D grid of the three tile kernels: workgroup w runs on XCD w % 8, and all
// 128-position tiles of one (batch, head) unit go to the same XCD, so that its L2 serves the K / V
// (Q / dO in the dK/dV kernel) reads of the unit's second and later tiles; heads cycle fastest over the
// units, so an XCD also sees only H / 8 (or one) of the bias planes.
struct AttnWg { int tile, h, b; bool ok; };
PE_DEV AttnWg attn_decode_wg(const AttnArgs& a) {
  const int nt = (a.L + 127) / 128;
  const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int u = (j / nt) * 8 + xcd;
  AttnWg r;
  r.tile = j % nt;
  r.ok = u < a.B * a.H;
  r.h = u % a.H;
  r.b = u / a.H;
  return r;
}
static inline unsigned attn_grid_size(long long B, int H, long long L) {
  const long long nt = (L + 127) / 128, units = B * H;
  return (unsigned)(8 * ((units + 7) / 8) * nt);
}

template <typename T> struct AttnCfg {
  static constexpr int VEC = Vec16<T>::N;
  static constexpr int KT = 64;                                   // positions staged per iteration
  static constexpr int RM = (sizeof(T) == 2) ? 40 : 36;           // row-major LDS row stride (elements), d padded <= 32
  static constexpr int TS = KT + 4;                               // transposed LDS row stride
};

PE_DEV int round_up_i(int a, int b) { return (a + b - 1) / b * b; }

// Stage `KT` rows (positions pos0..pos0+KT-1) of one [d]-vector per row into LDS, as a
// row-major copy (stride RM, columns d..DP-1 zero filled) and/or a transposed copy
// (rows = channel, stride TS).  Rows beyond L are zero.
template <typename T>
PE_DEV void attn_stage(const T* src /* at (w, h, b, position 0, 0) */, int seq_stride, int pos0, int L, int d, int DP,
                       T* lds_rm, T* lds_t, int tid, int nthreads) {
  typedef AttnCfg<T> C;
  typedef typename Vec16<T>::type V;
  const int vpr = DP / C::VEC;
  for (int idx = tid; idx < C::KT * vpr; idx += nthreads) {
    int row = idx / vpr, dd0 = (idx % vpr) * C::VEC;
    V v;
#pragma unroll
    for (int e = 0; e < C::VEC; e++) v[e] = from_f<T>(0.0f);
    int pos = pos0 + row;
    if (pos < L && dd0 < d) v = *reinterpret_cast<const V*>(src + pos * seq_stride + dd0);
    if (lds_rm) *reinterpret_cast<V*>(lds_rm + row * C::RM + dd0) = v;
    if (lds_t) {
#pragma unroll
      for (int e = 0; e < C::VEC; e++) lds_t[(dd0 + e) * C::TS + row] = v[e];
    }
  }
}

// The same staging in two halves, so that the global loads of the next tile can be in flight while
// the current one is being used: `load` fills up to two 16-byte vectors per thread (zero beyond L / d),
// `store` writes them to the row-major and / or transposed LDS copies.
template <typename T> struct AttnStageRegs { typename Vec16<T>::type v[2]; };
template <typename T>
PE_DEV void attn_stage_load(const T* src, int seq_stride, int pos0, int L, int d, int DP, AttnStageRegs<T>& r, int tid) {
  typedef AttnCfg<T> C;
  typedef typename Vec16<T>::type V;
  const int vpr = DP / C::VEC;
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int idx = tid + i * 256;
    V v;
#pragma unroll
    for (int e = 0; e < C::VEC; e++) v[e] = from_f<T>(0.0f);
    const int row = idx / vpr, dd0 = (idx % vpr) * C::VEC;
    const int pos = pos0 + row;
    if (idx < C::KT * vpr && pos < L && dd0 < d) v = *reinterpret_cast<const V*>(src + pos * seq_stride + dd0);
    r.v[i] = v;
  }
}
template <typename T>
PE_DEV void attn_stage_store(const AttnStageRegs<T>& r, int DP, T* lds_rm, T* lds_t, int tid) {
  typedef AttnCfg<T> C;
  typedef typename Vec16<T>::type V;
  const int vpr = DP / C::VEC;
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int idx = tid + i * 256;
    if (idx < C::KT * vpr) {
      const int row = idx / vpr, dd0 = (idx % vpr) * C::VEC;
      if (lds_rm) *reinterpret_cast<V*>(lds_rm + row * C::RM + dd0) = r.v[i];
      if (lds_t) {
#pragma unroll
        for (int e = 0; e < C::VEC; e++) lds_t[(dd0 + e) * C::TS + row] = r.v[i][e];
      }
    }
  }
}

// accumulator elements [u*KP, u*KP+KP) of a 32x32 tile as an MFMA operand fragment
template <typename T> PE_DEV typename Mma<T>::frag acc_to_frag(const f32x16& acc, int u);
template <> PE_DEV Mma<bf16>::frag acc_to_frag<bf16>(const f32x16& acc, int u) {
  bf16x8 f;
#pragma unroll
  for (int t = 0; t < 8; t++) f[t] = (bf16)acc[u * 8 + t];
  return f;
}
template <> PE_DEV Mma<float>::frag acc_to_frag<float>(const f32x16& acc, int u) { return acc[u]; }

// matching fragment of the other operand from a transposed LDS tile: row pointer `rowp`
// points at element [row = lane%32][tile_base]; contraction slots follow acc_row(g, a).
template <typename T> PE_DEV typename Mma<T>::frag lds_tfrag(const T* rowp, int g, int u);
template <> PE_DEV Mma<bf16>::frag lds_tfrag<bf16>(const bf16* rowp, int g, int u) {
  bf16x4 lo = *reinterpret_cast<const bf16x4*>(rowp + 16 * u + 4 * g);
  bf16x4 hi = *reinterpret_cast<const bf16x4*>(rowp + 16 * u + 8 + 4 * g);
  bf16x8 f;
  f[0] = lo[0]; f[1] = lo[1]; f[2] = lo[2]; f[3] = lo[3];
  f[4] = hi[0]; f[5] = hi[1]; f[6] = hi[2]; f[7] = hi[3];
  return f;
}
template <> PE_DEV Mma<float>::frag lds_tfrag<float>(const float* rowp, int g, int u) {
  return rowp[8 * (u >> 2) + 4 * g + (u & 3)];
}

// The same fragment from a ROW-major LDS tile [position][STRIDE] (bf16, transposing reads): channel l32, the 16 positions from
// pos0 in the order of acc_row.  No second, transposed copy, whose 2-byte stores were 8 per 16-byte vector.
template <int STRIDE> PE_DEV bf16x8 lds_rfrag(const bf16* tile, int pos0, int l32, int g) {
  const bf16* q = tile + (pos0 + 4 * g + ((l32 & 15) >> 2)) * STRIDE + (l32 & 16) + 4 * (l32 & 3);
  const bf16x4 lo = lds_read_tr(q), hi = lds_read_tr(q + 8 * STRIDE);
  bf16x8 f;
#pragma unroll
  for (int e = 0; e < 4; e++) { f[e] = lo[e]; f[4 + e] = hi[e]; }
  return f;
}
// a lane's position (row) of a [position][d] tensor from a transposed 32 x 32 accumulator tile, times f
template <typename T> PE_DEV void attn_store_row(T* row, const f32x16& acc, float f, int d, int g) {
  if constexpr (sizeof(T) == 2) {
    if (d % 8 == 0) {
#pragma unroll
      for (int j = 0; j < 2; j++) {
        float v[8];
        rows_unpack(acc, j, v);      // every lane of the wave takes part
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] *= f;
        bf16x8 t;
#pragma unroll
        for (int e = 0; e < 8; e++) t[e] = (bf16)v[e];
        if (row && 16 * j + 8 * g < d) *reinterpret_cast<bf16x8*>(row + 16 * j + 8 * g) = t;
      }
      return;
    }
  }
#pragma unroll
  for (int q4 = 0; q4 < 4; q4++) {
    const int dd = 8 * q4 + 4 * g;
    if (row && dd < d) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; r++) v[r] = acc[q4 * 4 + r] * f;
      store4<T>(row + dd, v);
    }
  }
}

// operand fragment straight from global memory: row `p` (nullptr = out of range), channels
// [kk*KSTEP + g*KP, +KP), zero beyond d
template <typename T> PE_DEV typename Mma<T>::frag gl_frag(const T* p, int kk, int g, int d) {
  typedef Mma<T> MM;
  int c0 = kk * MM::KSTEP + g * MM::KP;
  if (p == nullptr || c0 >= d) return MM::zero();
  return MM::load(p + c0);
}

// Softmax is evaluated in the base-2 domain: t = q' k + bias', p = 2^(t - m), where q' = q * log2 e / sqrt(d) comes out
// of the projection GEMM already scaled (its prepared weight copy carries the factor) and bias' = bias * log2 e is what
// bias_tile_kernel stores.  A logit costs the vector unit no multiply-add and no conversion:
//   * the bias tile is added by the matrix unit, as I x bias with an identity A operand (bf16; the 32-bit path adds it
//     with 16 vector adds), and is loaded in exactly the B-operand order, so it needs no conversion;
//   * the additive 0 / -inf key mask is applied only to 32-key tiles that hold a masked or padded key (one flag per
//     tile, decided when the tile is staged);
//   * in the dK / dV kernel, where -lse and -D of a tile's queries sit in LDS in accumulator order, they are the C
//     operands of the S and dP products.
// At L = 256 these kernels are bound by the length of a workgroup's life (memory round trips and dependent stages in a row
// at 3-4 waves per SIMD), not by any one unit: measured on MI355X, halving the vector instructions per logit changed the
// forward kernel by 2 %, taking the exponentials out by 3 %, while its loads and stores add their full time to the
// arithmetic's.  What helps is fewer round trips in a row (K / V staged 256 keys at a time in the forward kernel) and
// registers kept at the 128 that four waves per SIMD allow.
#define PE_LOG2E 1.4426950408889634f
#define PE_LN2 0.6931471805599453f
// raw v_exp_f32 (2^x; results below the normal range flush to zero, which is what softmax wants)
PE_DEV float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <typename T> PE_DEV f32x16 mma_c(typename Mma<T>::frag a, typename Mma<T>::frag b, const f32x16& c);
template <> PE_DEV f32x16 mma_c<bf16>(bf16x8 a, bf16x8 b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
template <> PE_DEV f32x16 mma_c<float>(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
PE_DEV f32x16 splat16(float v) {
  f32x16 r;
#pragma unroll
  for (int e = 0; e < 16; e++) r[e] = v;
  return r;
}

// Bias values of one 32x32 tile for the lane that owns position `col` (clamped to L-1 by the caller) of the lane axis,
// from the chunk-ordered plane of its head (bias_tile_kernel).  bf16: chunk c of lane group g holds positions
// 16 c + 8 g + 0..7 of the other axis, i.e. the B operand of MFMA step c; fp32: accumulator order.  16-byte loads; a half
// wave's 32 lanes read 512 contiguous bytes per load.  p: the lane's own address of chunk 0; chunks are 2 L lanes apart.
template <typename T> struct BiasTile;
template <> struct BiasTile<bf16> { bf16x8 v[2]; };
template <> struct BiasTile<float> { float v[16]; };
PE_DEV void attn_load_bias_at(const bf16* p, int L, BiasTile<bf16>& b) {
#pragma unroll
  for (int c = 0; c < 2; c++) b.v[c] = *reinterpret_cast<const bf16x8*>(p + (long long)c * 2 * L * BiasChunk<bf16>::CH);
}
PE_DEV void attn_load_bias_at(const float* p, int L, BiasTile<float>& b) {
#pragma unroll
  for (int c = 0; c < 4; c++) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + (long long)c * 2 * L * BiasChunk<float>::CH);
#pragma unroll
    for (int r = 0; r < 4; r++) b.v[c * 4 + r] = v[r];
  }
}
// identity A operand: lane (row l32, group g) of step c holds [16 c + 8 g + t == l32], t = 0..7
template <typename T> struct IdFrag;
template <> struct IdFrag<bf16> {
  bf16x8 f[2];
  PE_DEV void init(int l32, int g) {
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
      for (int t = 0; t < 8; t++) f[c][t] = (bf16)((16 * c + 8 * g + t == l32) ? 1.0f : 0.0f);
  }
};
template <> struct IdFrag<float> { PE_DEV void init(int, int) {} };
PE_DEV void attn_add_bias(f32x16& acc, const BiasTile<bf16>& b, const IdFrag<bf16>& id) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(id.f[0], b.v[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(id.f[1], b.v[1], acc, 0, 0, 0);
}
PE_DEV void attn_add_bias(f32x16& acc, const BiasTile<float>& b, const IdFrag<float>&) {
#pragma unroll
  for (int e = 0; e < 16; e++) acc[e] += b.v[e];
}
// additive key mask of one tile in accumulator order (rows of the tile = keys)
PE_DEV void attn_add_row_mask(f32x16& acc, const float* lds_madd_tile, int g) {
#pragma unroll
  for (int q4 = 0; q4 < 4; q4++) {
    const f32x4 ma = *reinterpret_cast<const f32x4*>(lds_madd_tile + 8 * q4 + 4 * g);
#pragma unroll
    for (int r = 0; r < 4; r++) acc[q4 * 4 + r] += ma[r];
  }
}
// Key mask of the 64 staged keys: lds_madd = 0 / -inf per key, lds_flag[t] = 1 when tile t holds a masked or padded
// key.  Called by threads 0..63 (one wave) with their key's mask value (0 beyond L).
PE_DEV void attn_stage_mask(float mk, float* lds_madd, int* lds_flag, int t64) {
  const bool masked = !(mk > 0.0f);
  lds_madd[t64] = masked ? -INFINITY : 0.0f;
  const unsigned long long bal = __ballot(masked);
  if (t64 == 0) { lds_flag[0] = (bal & 0xffffffffull) != 0; lds_flag[1] = (bal >> 32) != 0; }
}
// a lane's 16 elements of a score tile (dS) stored in the same chunk order, from its address of chunk 0
template <typename T> PE_DEV void attn_store_tile16_at(T* p, int L, const float (&v)[16]);
template <> PE_DEV void attn_store_tile16_at<float>(float* p, int L, const float (&v)[16]) {
#pragma unroll
  for (int c = 0; c < 4; c++) {
    float t[4];
#pragma unroll
    for (int r = 0; r < 4; r++) t[r] = v[c * 4 + r];
    store4<float>(p + (long long)c * 2 * L * BiasChunk<float>::CH, t);
  }
}
template <> PE_DEV void attn_store_tile16_at<bf16>(bf16* p, int L, const float (&v)[16]) {
#pragma unroll
  for (int c = 0; c < 2; c++) {
    bf16x8 o;   // non-temporal: read once, by the reduction over the batch axis
#pragma unroll
    for (int r = 0; r < 8; r++) o[r] = (bf16)v[c * 8 + r];
    __builtin_nontemporal_store(o, reinterpret_cast<bf16x8*>(p + (long long)c * 2 * L * BiasChunk<bf16>::CH));
  }
}
// number of 32-position tiles of an axis of length L
PE_DEV int attn_tiles32(int L) { return (L + 31) >> 5; }

// ---------------------------------------------------------------------------
// Forward
// grid attn_grid_size(B, H, L), 256 threads; wave w owns queries q0 = tile*128 + 32*w
// ---------------------------------------------------------------------------
// The running maximum is a REFERENCE m_ref that follows the true maximum only when it has to.  The first tile in which a
// query meets a finite logit sets m_ref to that tile's maximum (so a query with a single valid key gets the
// probability 1 and its value row back exactly); after that the probabilities 2^(t - m_ref) <= 2^TAU are used as they
// are, and only when a lane's tile maximum is more than TAU above m_ref the wave re-bases (accumulators and sum times
// 2^(old - new)).  The result o = acc / l and lse = (m_ref + log2 l) ln 2 do not depend on the reference.
#define ATTN_TAU 8.0f
// Forward: K and V are staged a CHUNK of up to 256 keys at a time: all loads of the chunk are issued at once and waited
// for once (with 64-key tiles a workgroup paid one memory round trip per tile, four to six in a row), and the waves then
// run through its tiles without a barrier.  38 KB of LDS per workgroup, four workgroups per CU.
template <typename T> struct AttnChunk {
  static constexpr int CH = (sizeof(T) == 2) ? 256 : 128;          // keys per chunk
  static constexpr int TS = CH + 4;                                // transposed row stride
  static constexpr int NV = CH * (32 / Vec16<T>::N) / 256;         // 16-byte vectors per thread and tensor (4)
};
// all vectors of one [CH keys][d] chunk for this thread: vector idx = tid + 256 i <-> (row idx / vpr, channels
// (idx % vpr) VEC ..) with vpr = 32 / VEC vector slots per row whatever d is (slots beyond d stay zero)
template <typename T>
PE_DEV void attn_chunk_load(const T* src, int pos0, int L, int d, typename Vec16<T>::type (&r)[AttnChunk<T>::NV], int tid) {
  typedef typename Vec16<T>::type V;
  constexpr int VEC = Vec16<T>::N;
  constexpr int vpr = 32 / VEC;
#pragma unroll
  for (int i = 0; i < AttnChunk<T>::NV; i++) {
    const int idx = tid + i * 256;
    V v;
#pragma unroll
    for (int e = 0; e < VEC; e++) v[e] = from_f<T>(0.0f);
    const int row = idx / vpr, dd0 = (idx % vpr) * VEC;
    const int pos = pos0 + row;
    if (pos < L && dd0 < d) v = *reinterpret_cast<const V*>(src + (long long)pos * d + dd0);
    r[i] = v;
  }
}
template <typename T>
PE_DEV void attn_chunk_store(const typename Vec16<T>::type (&r)[AttnChunk<T>::NV], int DP, T* lds_rm, T* lds_t, int tid) {
  typedef typename Vec16<T>::type V;
  constexpr int VEC = Vec16<T>::N;
  constexpr int vpr = 32 / VEC;
#pragma unroll
  for (int i = 0; i < AttnChunk<T>::NV; i++) {
    const int idx = tid + i * 256;
    const int row = idx / vpr, dd0 = (idx % vpr) * VEC;
    if (dd0 < DP) {
      if (lds_rm) *reinterpret_cast<V*>(lds_rm + row * AttnCfg<T>::RM + dd0) = r[i];
      if (lds_t) {
#pragma unroll
        for (int e = 0; e < VEC; e++) lds_t[(dd0 + e) * AttnChunk<T>::TS + row] = r[i][e];
      }
    }
  }
}

#ifndef PE_FWD_WAVES
#define PE_FWD_WAVES 4
#endif
// NK: contraction steps of the score products when known at compile time (bf16: 1 up to d = 16, 2 above), 0: from d.
// What bounds it: the vector unit, about 9 instructions per logit at d = 32 of which one is an exponential of four times the
// length (busy 0.51 of the time at L = 256, where a workgroup's life is short, 0.70 to 0.81 at 384 and 512, 0.88 at d = 8).  Hence no transposed copy of V, the partner's maximum by a lane swap instead of through LDS, a bias pointer that
// steps by a constant; outputs and gate pass through LDS at the end (64-byte runs; a query per lane is a 16-byte access per row).
template <typename T, bool HAS_BIAS, int NK = 0>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PE_FWD_WAVES, PE_FWD_WAVES))) void attn_fwd_kernel(AttnArgs a) {
  typedef AttnCfg<T> C;
  typedef Mma<T> MM;
  typedef AttnChunk<T> K;
  typedef typename Vec16<T>::type V;
  constexpr bool TR = sizeof(T) == 2;
  __shared__ __attribute__((aligned(16))) T lds_k[K::CH * C::RM];
  __shared__ __attribute__((aligned(16))) T lds_v[TR ? K::CH * 32 : 32 * K::TS];   // [key][32], or transposed [channel][key]
  __shared__ __attribute__((aligned(16))) float lds_madd[K::CH];   // 0 for a valid key, -inf for a masked one
  __shared__ int lds_flag[K::CH / 32];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5;
  const AttnWg wg = attn_decode_wg(a);
  if (!wg.ok) return;
  const int h = wg.h, b = wg.b;
  const int L = a.L, d = a.d;
  const int DP = round_up_i(d, MM::KSTEP);
  const int NKK = NK > 0 ? NK : DP / MM::KSTEP;
  const int q0 = wg.tile * 128 + wave * 32, qi = q0 + l32;       // this lane's query
  const bool qok = qi < L;
  const long long HP = (long long)a.H * a.plane;            // distance between the q, k, v, gate groups
  const T* base = (const T*)a.qkvg + h * a.plane + (long long)b * L * d;
  const T* qrow = qok ? base + qi * d : nullptr;

  constexpr int MAXKK = NK > 0 ? NK : 32 / MM::KSTEP;   // d <= 32
  typename MM::frag qf[MAXKK];
  f32x16 oacc = splat16(0.0f);
  float m_ref = 0.0f, l_part = 0.0f;     // l_part: this lane's keys only; the two halves of a query are added at the end
  float limit = -INFINITY;               // re-base above it: m_ref + TAU once a finite logit has been seen
  constexpr bool has_bias = HAS_BIAS;
  const int ntile = attn_tiles32(L);
  // this lane's bias chunks of the current tile; a tile further is a constant number of elements further
  constexpr int BCH = BiasChunk<T>::CH;
  const T* bptr = has_bias ? (const T*)a.biasQ + (long long)h * ntile * L * 32 + ((long long)g * L + min(qi, L - 1)) * BCH : nullptr;
  const long long bstep = (long long)L * 32;
  IdFrag<T> idf;
  idf.init(l32, g);
  int tile = 0;

  for (int c0 = 0; c0 < L; c0 += K::CH) {
    {
      V rk[K::NV], rv[K::NV];
      if (c0 > 0) __syncthreads();
      attn_chunk_load<T>(base + HP, c0, L, d, rk, tid);
      attn_chunk_load<T>(base + 2 * HP, c0, L, d, rv, tid);
      const int j = c0 + tid;
      const float mk = (tid < K::CH && j < L) ? a.mask[(long long)b * a.mask_bs + (long long)j * a.mask_ks] : 0.0f;
      if (c0 == 0) {
#pragma unroll
        for (int kk = 0; kk < MAXKK; kk++)
          if (kk < NKK) qf[kk] = gl_frag<T>(qrow, kk, g, d);
      }
      attn_chunk_store<T>(rk, DP, lds_k, (T*)nullptr, tid);
      if constexpr (TR) {
#pragma unroll
        for (int i = 0; i < K::NV; i++) *reinterpret_cast<V*>(lds_v + (tid + i * 256) * C::VEC) = rv[i];   // rows of 32, zeros beyond d
      } else {
        attn_chunk_store<T>(rv, DP, (T*)nullptr, lds_v, tid);
      }
      if (tid < K::CH) attn_stage_mask(mk, lds_madd + 64 * wave, lds_flag + 2 * wave, lane);
      __syncthreads();
    }
    const int jend = min(K::CH, L - c0);
    BiasTile<T> bt;
    if (has_bias) attn_load_bias_at(bptr, L, bt);
    for (int js = 0; js < jend; js += 32, tile++) {
      const int masked = __builtin_amdgcn_readfirstlane(lds_flag[js >> 5]);
      // base-2 logits for (query = lane, keys = acc rows)
      f32x16 sacc = splat16(0.0f);
      typename MM::frag kf[NK > 0 ? NK : 1];
      if constexpr (NK > 0) {
#pragma unroll
        for (int kk = 0; kk < NK; kk++) kf[kk] = MM::load(lds_k + (js + l32) * C::RM + kk * MM::KSTEP + g * MM::KP);
#pragma unroll
        for (int kk = 0; kk < NK; kk++) MM::mma(sacc, kf[kk], qf[kk]);
      } else {
#pragma unroll
        for (int kk = 0; kk < MAXKK; kk++)
          if (kk < NKK) MM::mma(sacc, MM::load(lds_k + (js + l32) * C::RM + kk * MM::KSTEP + g * MM::KP), qf[kk]);
      }
      if (has_bias) {
        attn_add_bias(sacc, bt, idf);
        if (tile + 1 < ntile) bptr += bstep;
        attn_load_bias_at(bptr, L, bt);   // next tile's bias
      }
      if (masked) attn_add_row_mask(sacc, lds_madd + js, g);
      float tmax = sacc[0];
#pragma unroll
      for (int e = 1; e < 16; e++) tmax = fmaxf(tmax, sacc[e]);
      tmax = pair_max(tmax);
      // re-base when the tile's maximum is more than TAU above the reference, and at the first finite logit (nothing is
      // accumulated before it)
      const bool rebase = tmax > limit;
      if (__any(rebase)) {
        const float m_new = rebase ? tmax : m_ref;
        const float corr = rebase && limit == -INFINITY ? 0.0f : fast_exp2(m_ref - m_new);
        if (rebase) limit = tmax + ATTN_TAU;
        m_ref = m_new;
        l_part *= corr;
#pragma unroll
        for (int e = 0; e < 16; e++) oacc[e] *= corr;
      }
      float psum = 0.0f;
#pragma unroll
      for (int e = 0; e < 16; e++) {
        float p = fast_exp2(sacc[e] - m_ref);
        sacc[e] = p;
        psum += p;
      }
      l_part += psum;
      // O^T[dd, i] += sum_j V^T[dd, j] P^T[j, i]
      if constexpr (TR) {
#pragma unroll
        for (int u = 0; u < 2; u++) MM::mma(oacc, lds_rfrag<32>(lds_v, js + 16 * u, l32, g), acc_to_frag<T>(sacc, u));
      } else {
        const T* vrow = lds_v + l32 * K::TS + js;
#pragma unroll
        for (int u = 0; u < 32 / MM::KSTEP; u++) MM::mma(oacc, lds_tfrag<T>(vrow, g, u), acc_to_frag<T>(sacc, u));
      }
    }
  }
  const float l_run = l_part + __shfl_xor(l_part, 32, 64);
  const float inv = (l_run > 0.0f) ? 1.0f / l_run : 0.0f;
  if (qok && g == 0 && a.lse) a.lse[((long long)b * a.H + h) * L + qi] = (l_run > 0.0f) ? (m_ref + log2f(l_run)) * PE_LN2 : 0.0f;
  if constexpr (TR) {
    if (d == 32) {
      __syncthreads();   // lds_k becomes the waves' pieces
      RowsPiece pc;
      pc.init(reinterpret_cast<bf16*>(lds_k) + wave * 1024, lane);
      const long long wrow = h * a.plane + ((long long)b * L + q0) * 32 + lane * 8;     // memory layout: 16 rows further is 512 elements further
      const bool ok0 = q0 + (lane >> 2) < L, ok1 = q0 + (lane >> 2) + 16 < L;
      bf16x8 gm[2], gf[2], of[2], ogf[2], t0, t1;
      const T* pg = (const T*)a.qkvg + 3 * HP + wrow;
      gm[0] = *reinterpret_cast<const bf16x8*>(ok0 ? pg : (const T*)a.qkvg);
      gm[1] = *reinterpret_cast<const bf16x8*>(ok1 ? pg + 512 : (const T*)a.qkvg);
      pc.to_frag(gm, gf[0], gf[1]);
#pragma unroll
      for (int j = 0; j < 2; j++) {
        float v[8];
        rows_unpack(oacc, j, v);
#pragma unroll
        for (int e = 0; e < 8; e++) {
          v[e] *= inv;
          of[j][e] = (bf16)v[e];
          ogf[j][e] = (bf16)(v[e] * sigmoidf_((float)gf[j][e]));
        }
      }
      pc.to_mem(ogf, t0, t1);
      if (ok0) *reinterpret_cast<bf16x8*>((T*)a.og + wrow) = t0;
      if (ok1) *reinterpret_cast<bf16x8*>((T*)a.og + wrow + 512) = t1;
      if (a.o) {
        pc.to_mem(of, t0, t1);
        if (ok0) *reinterpret_cast<bf16x8*>((T*)a.o + wrow) = t0;
        if (ok1) *reinterpret_cast<bf16x8*>((T*)a.o + wrow + 512) = t1;
      }
      return;
    }
  }
  if (!qok) return;
  const long long orow = h * a.plane + ((long long)b * L + qi) * d;
  T* po = a.o ? (T*)a.o + orow : nullptr;
  T* pog = (T*)a.og + orow;
  const T* pg = qrow + 3 * HP;
#pragma unroll
  for (int q4 = 0; q4 < 4; q4++) {
    int dd = 8 * q4 + 4 * g;
    if (dd < d) {
      float gv[4], ov[4], ogv[4];
      load4<T>(pg + dd, gv);
#pragma unroll
      for (int r = 0; r < 4; r++) {
        ov[r] = oacc[q4 * 4 + r] * inv;
        ogv[r] = ov[r] * sigmoidf_(gv[r]);
      }
      if (po) store4<T>(po + dd, ov);
      store4<T>(pog + dd, ogv);
    }
  }
}
template <typename T>
static inline void launch_attn_fwd(hipStream_t st, const AttnArgs& a) {
  const dim3 grid(attn_grid_size(a.B, a.H, a.L)), block(256);
#define PE_ATTN_FWD(NK)                                                                                   \
  do {                                                                                                    \
    if (a.biasQ) hipLaunchKernelGGL((attn_fwd_kernel<T, true, NK>), grid, block, 0, st, a);               \
    else hipLaunchKernelGGL((attn_fwd_kernel<T, false, NK>), grid, block, 0, st, a);                      \
  } while (0)
  if constexpr (sizeof(T) == 2) {
    if (a.d <= 16) PE_ATTN_FWD(1); else PE_ATTN_FWD(2);
  } else {
    PE_ATTN_FWD(0);
  }
#undef PE_ATTN_FWD
}

// ---------------------------------------------------------------------------
// Backward, step 0: dO = dog * sigmoid(g); dg = dog * o * s(1-s) -> dqkvg gate slot;
// D = sum_c dO * o.  One thread per (b, p, h).
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_pre_kernel(AttnArgs a) {
  // 8 lanes per (h, b, p): lane `sub` owns channels [4*sub, 4*sub+4); consecutive groups walk
  // consecutive positions of one head plane (contiguous memory)
  long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int sub = gid & 7;
  long long idx = gid >> 3;
  const long long M = (long long)a.B * a.L;
  long long total = M * a.H;
  const bool ok = idx < total;
  if (!ok) idx = total - 1;
  const int h = idx / M;
  const long long plin = idx % M;
  const int b = plin / a.L, p = plin % a.L;
  const int d = a.d;
  long long qoff = (3LL * a.H + h) * a.plane + plin * d;
  long long ooff = h * a.plane + plin * d;
  float Dsum = 0.0f;
  const int c0 = sub * 4;
  if (ok && c0 < d) {
    float gv[4], ov[4], dv[4], dov[4], dgv[4];
    load4<T>((const T*)a.qkvg + qoff + c0, gv);
    load4<T>((const T*)a.o + ooff + c0, ov);
    load4<T>((const T*)a.dog + ooff + c0, dv);
#pragma unroll
    for (int e = 0; e < 4; e++) {
      float sg = sigmoidf_(gv[e]);
      dov[e] = to_f(from_f<T>(dv[e] * sg));
      dgv[e] = dv[e] * ov[e] * sg * (1.0f - sg);
      Dsum += dov[e] * ov[e];
    }
    store4<T>((T*)a.dO + ooff + c0, dov);
    store4<T>((T*)a.dqkvg + qoff + c0, dgv);
  }
  Dsum += __shfl_xor(Dsum, 4, 64);
  Dsum += __shfl_xor(Dsum, 2, 64);
  Dsum += __shfl_xor(Dsum, 1, 64);
  if (ok && sub == 0) a.D[((long long)b * a.H + h) * a.L + p] = Dsum;
}

// ---------------------------------------------------------------------------
// Backward, dQ of an attention without a bias (one with a bias: attn_bwd_dq2_kernel).  Same tiling as the forward kernel.
// ---------------------------------------------------------------------------
// Capped at 128 registers (4 waves per SIMD instead of 3 at the 138 the compiler would take; three
// dwords spill): measured 85 -> 77 us per biased attention at L = 256.
template <typename T, int NK = 0>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void attn_bwd_dq_kernel(AttnArgs a) {
  typedef AttnCfg<T> C;
  typedef Mma<T> MM;
  __shared__ __attribute__((aligned(16))) T lds_k[C::KT * C::RM];
  __shared__ __attribute__((aligned(16))) T lds_kt[sizeof(T) == 2 ? 8 : 32 * C::TS];
  __shared__ __attribute__((aligned(16))) T lds_v[C::KT * C::RM];
  __shared__ __attribute__((aligned(16))) float lds_madd[C::KT];
  __shared__ int lds_flag[2];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5;
  const AttnWg wg = attn_decode_wg(a);
  if (!wg.ok) return;
  const int h = wg.h, b = wg.b;
  const int L = a.L, d = a.d;
  const int DP = round_up_i(d, MM::KSTEP);
  const int NKK = NK > 0 ? NK : DP / MM::KSTEP;
  const int qi = wg.tile * 128 + wave * 32 + l32;
  const bool qok = qi < L;
  const long long HP = (long long)a.H * a.plane;
  const T* base = (const T*)a.qkvg + h * a.plane + (long long)b * L * d;
  const T* qrow = qok ? base + qi * d : nullptr;
  const long long orow = h * a.plane + ((long long)b * L + qi) * d;
  const T* dorow = qok ? (const T*)a.dO + orow : nullptr;

  constexpr int MAXKK = NK > 0 ? NK : 32 / MM::KSTEP;
  constexpr bool TR = sizeof(T) == 2;     // the transposed fragments come from the row-major tile
  typename MM::frag qf[MAXKK], dof[MAXKK];
#pragma unroll
  for (int kk = 0; kk < MAXKK; kk++)
    if (kk < NKK) {
      qf[kk] = gl_frag<T>(qrow, kk, g, d);
      dof[kk] = gl_frag<T>(dorow, kk, g, d);
    }
  const long long sidx = ((long long)b * a.H + h) * L + qi;
  const float lse2 = qok ? a.lse[sidx] * PE_LOG2E : 0.0f;
  const float Di = qok ? a.D[sidx] : 0.0f;

  f32x16 dq;
#pragma unroll
  for (int e = 0; e < 16; e++) dq[e] = 0.0f;

  for (int j0 = 0; j0 < L; j0 += C::KT) {
    __syncthreads();
    attn_stage<T>(base + HP, d, j0, L, d, DP, lds_k, TR ? (T*)nullptr : lds_kt, tid, 256);
    attn_stage<T>(base + 2 * HP, d, j0, L, d, DP, lds_v, (T*)nullptr, tid, 256);
    if (tid < C::KT) {
      const int j = j0 + tid;
      attn_stage_mask((j < L) ? a.mask[(long long)b * a.mask_bs + (long long)j * a.mask_ks] : 0.0f, lds_madd, lds_flag, tid);
    }
    __syncthreads();
#pragma unroll
    for (int jt = 0; jt < C::KT / 32; jt++) {
      if (j0 + jt * 32 >= L) break;
      const int masked = __builtin_amdgcn_readfirstlane(lds_flag[jt]);
      const int off0 = (jt * 32 + l32) * C::RM + g * MM::KP;
      f32x16 sacc = splat16(0.0f), pacc = splat16(0.0f);
#pragma unroll
      for (int kk = 0; kk < MAXKK; kk++)
        if (kk < NKK) {
          MM::mma(sacc, MM::load(lds_k + off0 + kk * MM::KSTEP), qf[kk]);      // S^T = K Q^T
          MM::mma(pacc, MM::load(lds_v + off0 + kk * MM::KSTEP), dof[kk]);     // dP^T = V dO^T
        }
      if (masked) attn_add_row_mask(sacc, lds_madd + jt * 32, g);
#pragma unroll
      for (int e = 0; e < 16; e++) sacc[e] = fast_exp2(sacc[e] - lse2) * (pacc[e] - Di);     // dS = P (dP - D)
      if constexpr (TR) {
#pragma unroll
        for (int u = 0; u < 2; u++) MM::mma(dq, lds_rfrag<C::RM>(lds_k, jt * 32 + 16 * u, l32, g), acc_to_frag<T>(sacc, u));
      } else {
        const T* krow = lds_kt + l32 * C::TS + jt * 32;
#pragma unroll
        for (int u = 0; u < 32 / MM::KSTEP; u++) MM::mma(dq, lds_tfrag<T>(krow, g, u), acc_to_frag<T>(sacc, u));
      }
    }
  }
  attn_store_row<T>(qok ? (T*)a.dqkvg + orow : nullptr, dq, a.scale, d, g);
}

// ---------------------------------------------------------------------------
// Backward, dQ for TWO batch rows per workgroup (biased attention only).  Waves 0-3 work on batch row
// 2u, waves 4-7 on row 2u+1 of the same head and query tile, each group exactly as attn_bwd_dq_kernel
// with its own LDS tiles.  The bias gradient is a sum over the batch axis, so the two groups add their
// dS tiles before the write: the upper group passes each 32x32 tile through LDS (two buffers, one
// workgroup barrier per tile), the lower group adds its own and stores dS^T[u][h][key][query].  That
// halves the dS traffic and the input of the reduction that follows.  With an odd B the last
// workgroup's upper group runs on row B-1 again and contributes nothing.
// ---------------------------------------------------------------------------
#ifndef PE_DQ2_WAVES
#define PE_DQ2_WAVES 4
#endif
template <typename T, int NK = 0>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(PE_DQ2_WAVES, PE_DQ2_WAVES))) void attn_bwd_dq2_kernel(AttnArgs a) {
  typedef AttnCfg<T> C;
  typedef Mma<T> MM;
  __shared__ __attribute__((aligned(16))) T lds_k2[2][C::KT * C::RM];
  __shared__ __attribute__((aligned(16))) T lds_kt2[2][sizeof(T) == 2 ? 8 : 32 * C::TS];
  __shared__ __attribute__((aligned(16))) T lds_v2[2][C::KT * C::RM];
  __shared__ __attribute__((aligned(16))) float lds_madd2[2][C::KT];
  __shared__ int lds_flag2[2][2];
  __shared__ __attribute__((aligned(16))) float lds_x[2][4][16][64];   // [buffer][wave of the upper group][element][lane]

  const int tid = threadIdx.x, lane = tid & 63, wave8 = tid >> 6, l32 = lane & 31, g = lane >> 5;
  const int grp = wave8 >> 2, wave = wave8 & 3, tg = tid & 255;
  // XCD-aware decode as in attn_decode_wg, over (pair of batch rows, head) units
  const int nt = (a.L + 127) / 128, Bp = (a.B + 1) / 2;
  const int xcd = blockIdx.x & 7, jq = blockIdx.x >> 3;
  const int u = (jq / nt) * 8 + xcd;
  if (u >= Bp * a.H) return;
  const int tile = jq % nt, h = u % a.H, bp = u / a.H;
  const bool bvalid = 2 * bp + grp < a.B;
  const int b = bvalid ? 2 * bp + grp : a.B - 1;
  T* lds_k = lds_k2[grp];
  T* lds_kt = lds_kt2[grp];
  T* lds_v = lds_v2[grp];
  float* lds_madd = lds_madd2[grp];
  int* lds_flag = lds_flag2[grp];

  const int L = a.L, d = a.d;
  const int DP = round_up_i(d, MM::KSTEP);
  const int NKK = NK > 0 ? NK : DP / MM::KSTEP;
  const int qi = tile * 128 + wave * 32 + l32;
  const bool qok = qi < L;
  const long long HP = (long long)a.H * a.plane;
  const T* base = (const T*)a.qkvg + h * a.plane + (long long)b * L * d;
  const T* qrow = qok ? base + qi * d : nullptr;
  const long long orow = h * a.plane + ((long long)b * L + qi) * d;
  const T* dorow = qok ? (const T*)a.dO + orow : nullptr;

  constexpr int MAXKK = NK > 0 ? NK : 32 / MM::KSTEP;
  constexpr bool TR = sizeof(T) == 2;     // the transposed fragments come from the row-major tile
  typename MM::frag qf[MAXKK], dof[MAXKK];
#pragma unroll
  for (int kk = 0; kk < MAXKK; kk++)
    if (kk < NKK) {
      qf[kk] = gl_frag<T>(qrow, kk, g, d);
      dof[kk] = gl_frag<T>(dorow, kk, g, d);
    }
  const long long sidx = ((long long)b * a.H + h) * L + qi;
  const float lse2 = qok ? a.lse[sidx] * PE_LOG2E : 0.0f;
  const float Di = qok ? a.D[sidx] : 0.0f;
  // this lane's chunks of the current tile in the bias planes and (summed pair of rows, accumulator order) in the dS planes: the next
  // tile's are bstep elements further
  const int ntile = attn_tiles32(L);
  const long long bstep = (long long)L * 32, lane_off = ((long long)g * L + min(qi, L - 1)) * BiasChunk<T>::CH;
  const T* bptr = (const T*)a.biasQ + (long long)h * ntile * bstep + lane_off;
  T* dsptr = (T*)a.dS + ((long long)bp * a.H + h) * ntile * bstep + lane_off;
  IdFrag<T> idf;
  idf.init(l32, g);

  f32x16 dq;
#pragma unroll
  for (int e = 0; e < 16; e++) dq[e] = 0.0f;

  int xb = 0;   // exchange buffer of the current tile
  BiasTile<T> bt;
  attn_load_bias_at(bptr, L, bt);
  for (int j0 = 0; j0 < L; j0 += C::KT) {
    __syncthreads();
    attn_stage<T>(base + HP, d, j0, L, d, DP, lds_k, TR ? (T*)nullptr : lds_kt, tg, 256);
    attn_stage<T>(base + 2 * HP, d, j0, L, d, DP, lds_v, (T*)nullptr, tg, 256);
    if (tg < C::KT) {
      const int j = j0 + tg;
      attn_stage_mask((j < L) ? a.mask[(long long)b * a.mask_bs + (long long)j * a.mask_ks] : 0.0f, lds_madd, lds_flag, tg);
    }
    __syncthreads();
#pragma unroll
    for (int jt = 0; jt < C::KT / 32; jt++) {
      const int kt0 = j0 + jt * 32;
      if (kt0 >= L) break;   // uniform over the workgroup
      const int masked = __builtin_amdgcn_readfirstlane(lds_flag[jt]);
      const int off0 = (jt * 32 + l32) * C::RM + g * MM::KP;
      f32x16 sacc = splat16(0.0f), pacc = splat16(0.0f);
#pragma unroll
      for (int kk = 0; kk < MAXKK; kk++)
        if (kk < NKK) {
          MM::mma(sacc, MM::load(lds_k + off0 + kk * MM::KSTEP), qf[kk]);      // S^T = K Q^T
          MM::mma(pacc, MM::load(lds_v + off0 + kk * MM::KSTEP), dof[kk]);     // dP^T = V dO^T
        }
      attn_add_bias(sacc, bt, idf);
      if (kt0 + 32 < L) bptr += bstep;
      attn_load_bias_at(bptr, L, bt);   // next tile's bias
      if (masked) attn_add_row_mask(sacc, lds_madd + jt * 32, g);
#pragma unroll
      for (int e = 0; e < 16; e++) sacc[e] = fast_exp2(sacc[e] - lse2) * (pacc[e] - Di);     // dS = P (dP - D)
      // the upper group hands its dS tile over; the lower group adds its own and writes the sum
      if (grp == 1) {
#pragma unroll
        for (int e = 0; e < 16; e++) lds_x[xb][wave][e][lane] = bvalid ? sacc[e] : 0.0f;
      }
      __syncthreads();
      if (grp == 0 && qok) {   // 16-byte stores; a half wave's lanes write 512 contiguous bytes each
        float v16[16];
#pragma unroll
        for (int e = 0; e < 16; e++) v16[e] = sacc[e] + lds_x[xb][wave][e][lane];
        attn_store_tile16_at<T>(dsptr, L, v16);
      }
      xb ^= 1;
      dsptr += bstep;
      if constexpr (TR) {
#pragma unroll
        for (int uu = 0; uu < 2; uu++) MM::mma(dq, lds_rfrag<C::RM>(lds_k, jt * 32 + 16 * uu, l32, g), acc_to_frag<T>(sacc, uu));
      } else {
        const T* krow = lds_kt + l32 * C::TS + jt * 32;
#pragma unroll
        for (int uu = 0; uu < 32 / MM::KSTEP; uu++) MM::mma(dq, lds_tfrag<T>(krow, g, uu), acc_to_frag<T>(sacc, uu));
      }
    }
  }
  attn_store_row<T>(qok && bvalid ? (T*)a.dqkvg + orow : nullptr, dq, a.scale, d, g);
}

// ---------------------------------------------------------------------------
// Backward, dK and dV.  Wave w owns keys k0 = tile*128 + 32*w (a key is a lane);
// loops over query tiles staged in LDS (row-major and transposed copies of Q and dO).
// ---------------------------------------------------------------------------
#ifndef PE_DKV_WAVES
#define PE_DKV_WAVES 3
#endif
template <typename T, bool HAS_BIAS, int NK = 0>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PE_DKV_WAVES, PE_DKV_WAVES))) void attn_bwd_dkv_kernel(AttnArgs a) {
  typedef AttnCfg<T> C;
  typedef Mma<T> MM;
  __shared__ __attribute__((aligned(16))) T lds_q[C::KT * C::RM];
  __shared__ __attribute__((aligned(16))) T lds_qt[sizeof(T) == 2 ? 8 : 32 * C::TS];
  __shared__ __attribute__((aligned(16))) T lds_do[C::KT * C::RM];
  __shared__ __attribute__((aligned(16))) T lds_dot[sizeof(T) == 2 ? 8 : 32 * C::TS];
  __shared__ __attribute__((aligned(16))) float lds_lse[C::KT];   // minus the base-2 log-sum-exp, -inf beyond L
  __shared__ __attribute__((aligned(16))) float lds_D[C::KT];     // minus D

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5;
  const AttnWg wg = attn_decode_wg(a);
  if (!wg.ok) return;
  const int h = wg.h, b = wg.b;
  const int L = a.L, d = a.d;
  const int DP = round_up_i(d, MM::KSTEP);
  const int NKK = NK > 0 ? NK : DP / MM::KSTEP;
  const int kj = wg.tile * 128 + wave * 32 + l32;       // this lane's key
  const bool kok = kj < L;
  const long long HP = (long long)a.H * a.plane;
  const T* base = (const T*)a.qkvg + h * a.plane + (long long)b * L * d;
  const T* krow = kok ? base + HP + kj * d : nullptr;
  const T* vrow = kok ? base + 2 * HP + kj * d : nullptr;
  const T* dobase = (const T*)a.dO + h * a.plane + (long long)b * L * d;

  constexpr int MAXKK = NK > 0 ? NK : 32 / MM::KSTEP;
  constexpr bool TR = sizeof(T) == 2;     // the transposed fragments come from the row-major tile
  typename MM::frag kf[MAXKK], vf[MAXKK];
#pragma unroll
  for (int kk = 0; kk < MAXKK; kk++)
    if (kk < NKK) {
      kf[kk] = gl_frag<T>(krow, kk, g, d);
      vf[kk] = gl_frag<T>(vrow, kk, g, d);
    }
  const float mk = kok ? a.mask[(long long)b * a.mask_bs + (long long)kj * a.mask_ks] : 0.0f;
  const float madd = (mk > 0.0f) ? 0.0f : -INFINITY;
  const bool wave_masked = __any(!(mk > 0.0f));          // some key of this wave is masked or padded
  constexpr bool has_bias = HAS_BIAS;
  const int ntile = attn_tiles32(L);
  const long long bstep = (long long)L * 32;      // elements between this lane's bias chunks of neighbouring tiles
  const T* bptr = has_bias ? (const T*)a.biasK + (long long)h * ntile * bstep + ((long long)g * L + min(kj, L - 1)) * BiasChunk<T>::CH : nullptr;
  IdFrag<T> idf;
  idf.init(l32, g);

  f32x16 dk, dv;
#pragma unroll
  for (int e = 0; e < 16; e++) { dk[e] = 0.0f; dv[e] = 0.0f; }

  // Q, dO, -lse and -D of the next 64 queries are loaded into registers while the current ones are used; the bias
  // one 32-query tile ahead of its use
  AttnStageRegs<T> rq, rdo;
  float r_lse = 0.0f, r_D = 0.0f;
  auto prefetch = [&](int i0) {
    attn_stage_load<T>(base, d, i0, L, d, DP, rq, tid);
    attn_stage_load<T>(dobase, d, i0, L, d, DP, rdo, tid);
    const int i = i0 + tid;
    const bool ok = tid < C::KT && i < L;
    const long long sidx = ((long long)b * a.H + h) * L + (ok ? i : 0);
    r_lse = ok ? -a.lse[sidx] * PE_LOG2E : -INFINITY;
    r_D = ok ? -a.D[sidx] : 0.0f;
  };
  prefetch(0);
  BiasTile<T> bt;                       // refilled for the next 32-query tile as soon as its MFMAs have taken it
  if (has_bias) attn_load_bias_at(bptr, L, bt);
  for (int i0 = 0; i0 < L; i0 += C::KT) {
    __syncthreads();
    attn_stage_store<T>(rq, DP, lds_q, TR ? (T*)nullptr : lds_qt, tid);
    attn_stage_store<T>(rdo, DP, lds_do, TR ? (T*)nullptr : lds_dot, tid);
    if (tid < C::KT) { lds_lse[tid] = r_lse; lds_D[tid] = r_D; }
    __syncthreads();
    if (i0 + C::KT < L) prefetch(i0 + C::KT);
#pragma unroll
    for (int it = 0; it < C::KT / 32; it++) {
      if (i0 + it * 32 >= L) break;
      // C operands: -lse and -D of the tile's queries in accumulator order
      f32x16 sacc, pacc;
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const f32x4 ls = *reinterpret_cast<const f32x4*>(lds_lse + it * 32 + 8 * q4 + 4 * g);
        const f32x4 Dr = *reinterpret_cast<const f32x4*>(lds_D + it * 32 + 8 * q4 + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; r++) { sacc[q4 * 4 + r] = ls[r]; pacc[q4 * 4 + r] = Dr[r]; }
      }
#pragma unroll
      for (int kk = 0; kk < MAXKK; kk++)
        if (kk < NKK) {
          int off = (it * 32 + l32) * C::RM + kk * MM::KSTEP + g * MM::KP;
          MM::mma(sacc, MM::load(lds_q + off), kf[kk]);      // S - lse = Q K^T - lse   (rows queries, col = key lane)
          MM::mma(pacc, MM::load(lds_do + off), vf[kk]);     // dP - D = dO V^T - D
        }
      if (has_bias) {
        attn_add_bias(sacc, bt, idf);
        if ((i0 >> 5) + it + 1 < ntile) bptr += bstep;
        attn_load_bias_at(bptr, L, bt);
      }
      if (wave_masked) {
#pragma unroll
        for (int e = 0; e < 16; e++) sacc[e] += madd;
      }
      f32x16 pv;
#pragma unroll
      for (int e = 0; e < 16; e++) {
        const float p = fast_exp2(sacc[e]);
        pv[e] = p;
        sacc[e] = p * pacc[e];                                // dS = P (dP - D)
      }
      if constexpr (TR) {
#pragma unroll
        for (int u = 0; u < 2; u++) {
          MM::mma(dv, lds_rfrag<C::RM>(lds_do, it * 32 + 16 * u, l32, g), acc_to_frag<T>(pv, u));     // dV^T += dO^T P
          MM::mma(dk, lds_rfrag<C::RM>(lds_q, it * 32 + 16 * u, l32, g), acc_to_frag<T>(sacc, u));    // dK^T += Q^T dS
        }
      } else {
        const T* dotrow = lds_dot + l32 * C::TS + it * 32;
        const T* qtrow = lds_qt + l32 * C::TS + it * 32;
#pragma unroll
        for (int u = 0; u < 32 / MM::KSTEP; u++) {
          MM::mma(dv, lds_tfrag<T>(dotrow, g, u), acc_to_frag<T>(pv, u));
          MM::mma(dk, lds_tfrag<T>(qtrow, g, u), acc_to_frag<T>(sacc, u));
        }
      }
    }
  }
  T* pdk = kok ? (T*)a.dqkvg + HP + h * a.plane + ((long long)b * L + kj) * d : nullptr;
  attn_store_row<T>(pdk, dk, PE_LN2, d, g);                       // q' = q scale log2 e
  attn_store_row<T>(pdk ? pdk + HP : nullptr, dv, 1.0f, d, g);
}

// dQ (and dS, two batch rows per workgroup, for a biased attention)
template <typename T>
static inline void launch_attn_bwd_dq(hipStream_t st, const AttnArgs& a) {
  const long long B = a.biasQ ? (a.B + 1) / 2 : a.B;
  const dim3 grid(attn_grid_size(B, a.H, a.L));
#define PE_ATTN_DQ(NK)                                                                             \
  do {                                                                                             \
    if (a.biasQ) hipLaunchKernelGGL((attn_bwd_dq2_kernel<T, NK>), grid, dim3(512), 0, st, a);      \
    else hipLaunchKernelGGL((attn_bwd_dq_kernel<T, NK>), grid, dim3(256), 0, st, a);        \
  } while (0)
  if constexpr (sizeof(T) == 2) {
    if (a.d <= 16) PE_ATTN_DQ(1); else PE_ATTN_DQ(2);
  } else {
    PE_ATTN_DQ(0);
  }
#undef PE_ATTN_DQ
}
template <typename T>
static inline void launch_attn_bwd_dkv(hipStream_t st, const AttnArgs& a) {
  const dim3 grid(attn_grid_size(a.B, a.H, a.L)), block(256);
#define PE_ATTN_DKV(NK)                                                                            \
  do {                                                                                             \
    if (a.biasK) hipLaunchKernelGGL((attn_bwd_dkv_kernel<T, true, NK>), grid, block, 0, st, a);    \
    else hipLaunchKernelGGL((attn_bwd_dkv_kernel<T, false, NK>), grid, block, 0, st, a);           \
  } while (0)
  if constexpr (sizeof(T) == 2) {
    if (a.d <= 16) PE_ATTN_DKV(1); else PE_ATTN_DKV(2);
  } else {
    PE_ATTN_DKV(0);
  }
#undef PE_ATTN_DKV
}

// ---------------------------------------------------------------------------
// Backward of the biased attention at head dimension 8 over many batch rows (bf16): dQ, dK, dV and the bias gradient in
// one kernel.  A workgroup owns (head, 128 keys) and WALKS through the batch rows of its split; a wave owns 32 keys
// and up to four query tiles, whose dS sums over those rows stay in its registers until the end.
//
// At d = 8 a row's q, k, v, dO are 16 bytes per position while its 32 x 32 logit tiles cost as much as at d = 32: the
// separate dQ and dK / dV kernels evaluated every tile twice (vector unit), read a 96 KB bias slab per workgroup for 24 KB
// of operands, and passed the bias gradient through memory once per pair of batch rows.  Here a tile is evaluated
// once:
//   * scores with a key per lane (as in the dK / dV kernel): dK and dV are contractions over accumulator rows; they share
//     one accumulator (rows 0-7 dV, 8-15 dK: the A operands are [dO^T; 0] and [0; Q^T]);
//   * -lse, -D and the key mask are contraction slots 8..: at d = 8 half of the K = 16 MFMA step is free, so S - lse + mask
//     and dP - D come out of the matrix unit.  lse and D enter as three bf16 pieces each, 24 bits: exact in fp32;
//   * dS goes to LDS [query][key] in bf16, as which it is an operand of dQ anyway; after a barrier a wave contracts one query
//     tile with the workgroup's 128 keys.  With more than 128 keys dQ is a sum of fp32 partials per key block.
// 768 threads: 12 waves x 4 tiles are the 12 x 4 tiles of L = 384, three waves per SIMD leave 168 registers (64 of them
// the dS sums); 156 KB of LDS, one workgroup per CU.
// Measured at B = 5120, L = 384, H = 8: 3.13 ms + 0.34 ms for the dQ sum, before it dQ 3.7 + dK / dV 2.86 + reduction
// 0.85 ms; at B = 1024, L = 256: 0.30 ms instead of 0.83 ms.
struct AttnWalk {
  static constexpr int LMAX = 384, KB = 128, THREADS = 768, NTILE = 4;
  static constexpr int SD = KB + 8, ST = LMAX + 8;    // row strides of the dS and the transposed tiles
};
// x as a sum of three bf16 pieces in slots 0..2
PE_DEV void attn_split3(float x, bf16x8& v) {
  v[0] = (bf16)x;
  const float r1 = x - (float)v[0];
  v[1] = (bf16)r1;
  v[2] = (bf16)(r1 - (float)v[1]);
}
// 16 bytes at a uniform base and a 32-bit byte offset per lane: one address register
PE_DEV bf16x8 attn_ld8(const bf16* base, unsigned off) {
  return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(base) + off);
}
// grid H * ceil(L / 128) * nsplit.  dqp: fp32 [key block][H][B L][8], used when L > 128.  dSp: fp32 [nsplit][H] planes in the
// layout of dS.  Heads cycle fastest over the workgroups, i.e. over the XCDs, so an L2 holds the bias planes of few heads.
__global__ __launch_bounds__(AttnWalk::THREADS) void attn_bwd_walk_kernel(AttnArgs a, float* dqp, float* dSp, int nsplit) {
  typedef AttnWalk W;
  typedef Mma<bf16> MM;
  __shared__ __attribute__((aligned(16))) bf16 lds_ds[W::LMAX * W::SD];    // [query][key]
  __shared__ __attribute__((aligned(16))) bf16 lds_rm[2 * W::LMAX * 16];   // rows of q, then of dO: 8 channels, 8 extra slots
  __shared__ __attribute__((aligned(16))) bf16 lds_t[24 * W::ST];          // rows: dO^T (8), zeros (8), Q^T (8)
  __shared__ __attribute__((aligned(16))) bf16 lds_kv[2 * W::KB * 16];     // rows of K, then of V, with extra slots
  __shared__ __attribute__((aligned(16))) bf16 lds_kt[8 * W::SD];          // K^T
  __shared__ __attribute__((aligned(16))) bf16 lds_id[2 * 64 * 8];         // the identity operand of the bias step
  float* lds_x = reinterpret_cast<float*>(lds_rm);   // dK / dV of 8 waves, 16 KB: the rows are free by then

  // everything that is the same in a wave is in scalar registers: the vector registers are full
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int L = a.L, H = a.H, nqt = (L + 31) >> 5, nkb = (L + W::KB - 1) / W::KB;
  const int h = blockIdx.x % H, kb = (blockIdx.x / H) % nkb, split = blockIdx.x / (H * nkb);
  const int b0 = (int)((long long)split * a.B / nsplit), b1 = (int)((long long)(split + 1) * a.B / nsplit);
  const int kt = wave & 3, qg = wave >> 2;
  const int k0 = kb * W::KB;
  const bool kactive = k0 + kt * 32 < L;
  const int nks = min(W::KB / 16, ((L - k0 + 31) >> 5) * 2);   // 16-key steps of this key block
  const long long HP = (long long)H * a.plane;
  const bf16* qbase = (const bf16*)a.qkvg + h * a.plane;
  const bf16* dobase = (const bf16*)a.dO + h * a.plane;
  const bf16* bplane = (const bf16*)a.biasK + (long long)h * nqt * L * 32;
  unsigned boff = (unsigned)(g * L + min(k0 + kt * 32 + l32, L - 1)) * 16;   // this lane's place in a bias chunk, bytes
  // staging: thread tid < 384 brings q row tid, the others dO row tid - 384; threads 0..127 also a K row, 128..255 a V row
  const bool isq = wave < W::LMAX / 64, isk = wave < W::KB / 64, iskv = wave < 2 * W::KB / 64;
  unsigned srow = isq ? tid : tid - W::LMAX, krow = tid & (W::KB - 1);
  const bf16* const ssrc = isq ? qbase : dobase;
  const float* const fsrc = (isq ? a.lse : a.D) + (long long)h * L;
  const bf16* const ksrc = qbase + (isk ? HP : 2 * HP) + k0 * 8;
  const unsigned nkey = L - k0;
  bf16x8 sv, kv;
  float sf = 0.0f, mk = 0.0f;
#define PE_WALK_LOAD(b)                                                                                              \
  do {                                                                                                               \
    sv = MM::zero(); kv = MM::zero(); sf = 0.0f; mk = 0.0f;                                                          \
    if (srow < (unsigned)L) {                                                                                        \
      sv = attn_ld8(ssrc + (long long)(b) * L * 8, srow * 16u);                                                      \
      sf = (fsrc + (long long)(b) * H * L)[srow];                                                                    \
    }                                                                                                                \
    if (iskv && krow < nkey) {                                                                                       \
      kv = attn_ld8(ksrc + (long long)(b) * L * 8, krow * 16u);                                                      \
      if (isk) mk = a.mask[(long long)(b) * a.mask_bs + (long long)(k0 + krow) * a.mask_ks];                         \
    }                                                                                                                \
  } while (0)
// bias of query tile qt (uniform), as attn_load_bias_at
#define PE_WALK_BIAS(qt)                                                                                             \
  do {                                                                                                               \
    const bf16* tp = bplane + (long long)(qt) * L * 32;                                                              \
    asm volatile("" : "+v"(boff));   /* base + offset is not kept across the loop */                                 \
    bt.v[0] = attn_ld8(tp, boff);                                                                                    \
    bt.v[1] = attn_ld8(tp + (long long)L * 16, boff);                                                                \
  } while (0)

  if (wave == 0) {
    IdFrag<bf16> idf;
    idf.init(l32, g);
#pragma unroll
    for (int c = 0; c < 2; c++) *reinterpret_cast<bf16x8*>(lds_id + (c * 64 + lane) * 8) = idf.f[c];
  }
  for (int i = tid; i < 8 * W::ST; i += W::THREADS) lds_t[8 * W::ST + i] = (bf16)0.0f;
  f32x16 acc[W::NTILE];
#pragma unroll
  for (int t = 0; t < W::NTILE; t++) acc[t] = splat16(0.0f);
  BiasTile<bf16> bt;
  PE_WALK_BIAS(min(qg, nqt - 1));
  PE_WALK_LOAD(b0);

  for (int b = b0; b < b1; b++) {
    // per-lane indices anew for every row: their addresses would otherwise be kept in registers across the loop
    tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    lane = tid & 63; l32 = lane & 31; g = lane >> 5;
    srow = isq ? tid : tid - W::LMAX; krow = tid & (W::KB - 1);
    // ---- this row's operands to LDS ----
    if (srow < nqt * 32u) {
#pragma unroll
      for (int e = 0; e < 8; e++) lds_t[((isq ? 16 : 0) + e) * W::ST + srow] = sv[e];
    }
    if (iskv) {
      bf16x8 x = MM::zero();
      x[0] = x[1] = x[2] = (bf16)1.0f;
      if (isk) {
        x[3] = (bf16)((mk > 0.0f) ? 0.0f : -INFINITY);
#pragma unroll
        for (int e = 0; e < 8; e++) lds_kt[e * W::SD + krow] = kv[e];
      }
      *reinterpret_cast<bf16x8*>(lds_kv + tid * 16) = kv;
      *reinterpret_cast<bf16x8*>(lds_kv + tid * 16 + 8) = x;
    }
    __syncthreads();   // lds_x (the previous row's dK / dV) has been read
    if (srow < nqt * 32u) {
      bf16x8 x = MM::zero();
      if (srow < (unsigned)L) attn_split3(isq ? -sf * PE_LOG2E : -sf, x);
      else if (isq) x[0] = (bf16)-INFINITY;          // probability 0 for the queries beyond L
      if (isq) x[3] = (bf16)1.0f;                    // takes the key mask
      *reinterpret_cast<bf16x8*>(lds_rm + tid * 16) = sv;
      *reinterpret_cast<bf16x8*>(lds_rm + tid * 16 + 8) = x;
    }
    __syncthreads();
    if (b + 1 < b1) PE_WALK_LOAD(b + 1);

    // ---- score tiles: dS to registers (sum over rows) and LDS, dK and dV ----
    f32x16 dkv = splat16(0.0f);
    if (kactive) {
      const bf16x8 kf = MM::load(lds_kv + (kt * 32 + l32) * 16 + g * 8);
      const bf16x8 vf = MM::load(lds_kv + (W::KB + kt * 32 + l32) * 16 + g * 8);
#pragma unroll
      for (int t = 0; t < W::NTILE; t++) {
        const int qt = qg + 3 * t;
        if (qt < nqt) {
          const bf16* qrow = lds_rm + (qt * 32 + l32) * 16 + g * 8;
          f32x16 s = mma_c<bf16>(MM::load(qrow), kf, splat16(0.0f));                       // S - lse + mask
          f32x16 p = mma_c<bf16>(MM::load(qrow + W::LMAX * 16), vf, splat16(0.0f));        // dP - D
#pragma unroll
          for (int c = 0; c < 2; c++) s = mma_c<bf16>(MM::load(lds_id + (c * 64 + lane) * 8), bt.v[c], s);
          const int qn = qt + 3 < nqt && t + 1 < W::NTILE ? qt + 3 : qg;                   // next tile's bias
          PE_WALK_BIAS(qn);
#pragma unroll
          for (int e = 0; e < 16; e++) {
            s[e] = fast_exp2(s[e]);
            p[e] *= s[e];                                                                  // dS = P (dP - D)
            acc[t][e] += p[e];
          }
          const bf16* trow = lds_t + (l32 & 15) * W::ST + qt * 32;
          bf16* drow = lds_ds + (qt * 32 + 4 * g) * W::SD + kt * 32 + l32;
#pragma unroll
          for (int u = 0; u < 2; u++) {
            const bf16x8 sfr = acc_to_frag<bf16>(p, u);
            MM::mma(dkv, lds_tfrag<bf16>(trow, g, u), acc_to_frag<bf16>(s, u));            // dV^T += dO^T P
            MM::mma(dkv, lds_tfrag<bf16>(trow + 8 * W::ST, g, u), sfr);                    // dK^T += Q^T dS
#pragma unroll
            for (int e = 0; e < 8; e++) drow[(16 * u + 8 * (e >> 2) + (e & 3)) * W::SD] = sfr[e];
          }
        }
        __builtin_amdgcn_sched_barrier(0);   // one tile's operands at a time in registers
      }
    }
    __syncthreads();
    // ---- dK / dV partial sums of the waves that share keys; dQ of one query tile per wave ----
    if (qg > 0 && kactive) {
#pragma unroll
      for (int e = 0; e < 8; e++) lds_x[(((qg - 1) * 4 + kt) * 8 + e) * 64 + lane] = dkv[e];
    }
    if (wave < nqt) {
      const bf16* drow = lds_ds + (wave * 32 + l32) * W::SD + 8 * g;
      const bf16* ktrow = lds_kt + (l32 & 7) * W::SD + 8 * g;
      f32x16 dq = splat16(0.0f);
      for (int u = 0; u < nks; u++) MM::mma(dq, MM::load(ktrow + 16 * u), MM::load(drow + 16 * u));
      const int qi = wave * 32 + l32;
      if (qi < L) {
        const long long row = h * a.plane + ((long long)b * L + wave * 32) * 8;
        const unsigned off = l32 * 8 + 4 * g;
        float v[4];
        if (nkb == 1) {
#pragma unroll
          for (int r = 0; r < 4; r++) v[r] = dq[r] * a.scale;
          store4<bf16>((bf16*)a.dqkvg + row + off, v);
        } else {
#pragma unroll
          for (int r = 0; r < 4; r++) v[r] = dq[r];
          store4<float>(dqp + kb * HP + row + off, v);
        }
      }
    }
    __syncthreads();
    if (qg == 0 && k0 + kt * 32 + l32 < L) {
      float dv[4], dk[4];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        dv[r] = (dkv[r] + lds_x[(kt * 8 + r) * 64 + lane]) + lds_x[((4 + kt) * 8 + r) * 64 + lane];
        dk[r] = ((dkv[4 + r] + lds_x[(kt * 8 + 4 + r) * 64 + lane]) + lds_x[((4 + kt) * 8 + 4 + r) * 64 + lane]) * PE_LN2;   // q' = q scale log2 e
      }
      bf16* pdk = (bf16*)a.dqkvg + HP + h * a.plane + ((long long)b * L + k0 + kt * 32) * 8;
      const unsigned off = l32 * 8 + 4 * g;
      store4<bf16>(pdk + off, dk);
      store4<bf16>(pdk + HP + off, dv);
    }
  }
#undef PE_WALK_LOAD
#undef PE_WALK_BIAS
  if (!kactive) return;
  // this lane's key inside the chunk order of dS: accumulator element ek of lane group gk
  const int ek = 4 * (l32 >> 3) + (l32 & 3), gk = (l32 >> 2) & 1;
  float* dst = dSp + ((long long)split * H + h) * nqt * L * 32 + (ek & 7);
#pragma unroll
  for (int t = 0; t < W::NTILE; t++)
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int qi = (qg + 3 * t) * 32 + acc_row(g, e);
      if (qi < L) dst[bias_chunk_off<bf16>((k0 >> 5) + kt, ek >> 3, gk, qi, L)] = acc[t][e];
    }
}
// dQ = scale * sum of the fp32 partials of the key blocks; 8 channels per thread, n8 = H B L
__global__ __launch_bounds__(256) void attn_dq_sum_kernel(const float* dqp, bf16* dq, int nkb, long long n8, float scale) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n8) return;
  float s[8];
  ld8_once<float>(dqp + i * 8, s);
  for (int k = 1; k < nkb; k++) {
    float v[8];
    ld8_once<float>(dqp + (k * n8 + i) * 8, v);
#pragma unroll
    for (int e = 0; e < 8; e++) s[e] += v[e];
  }
#pragma unroll
  for (int e = 0; e < 8; e++) s[e] *= scale;
  st8<bf16>(dq + i * 8, s);
}
// Workgroups along the batch axis of attn_bwd_walk_kernel, 0: the call keeps the kernels per batch row.  A workgroup
// takes 32 rows or more (it writes one 32-bit dS plane for them) and two rounds of workgroups fill the CUs; below 128 workgroups half
// of the CUs would idle.  At the line both are close (B 256, L 256, one-stream block: 2.72 ms without, 2.71 ms with it);
// B 512, L 40: 1.03 -> 0.97 ms; B 5120, L 40: 2.77 -> 2.36 ms; B 1024, L 128: 1.99 -> 1.89 ms.  A last key
// block with one active key tile of four does not change that (one-stream blocks; L 136: B 1024 2.45 -> 2.27 ms, B 512 1.92 -> 1.82,
// B 256 1.54 -> 1.54; L 264: B 1024 5.16 -> 4.74, B 256 3.29 -> 3.19 ms).
static inline int attn_walk_splits(bool bf, bool bias, long long B, int H, long long L, int d) {
  if (!bf || !bias || d != 8 || L > AttnWalk::LMAX) return 0;
  const long long units = H * ((L + AttnWalk::KB - 1) / AttnWalk::KB);
  const long long n = std::min<long long>(B / 32, std::max<long long>(512 / units, 1));
  return n * units >= 128 ? (int)n : 0;
}

// The same reduction with 8 consecutive outputs per thread (16-byte loads for bf16) and eight loads in
// flight: 64 output groups x 4 batch lanes per workgroup.  Needs hll % 8 == 0 and 16-byte aligned buffers.
template <typename T>
__global__ __launch_bounds__(256) void attn_dbias_reduce8_kernel(const T* dS, float* dbias, int B, long long hll) {
  __shared__ float red[3][64][8];
  const int x = threadIdx.x & 63, y = threadIdx.x >> 6;
  const long long idx = ((long long)blockIdx.x * 64 + x) * 8;
  float s[8];
#pragma unroll
  for (int e = 0; e < 8; e++) s[e] = 0.0f;
  if (idx < hll) {
    for (int b = y; b < B; b += 32) {
      float v[8][8];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const int bb = b + 4 * u;
        if (bb < B) ld8_once<T>(dS + (long long)bb * hll + idx, v[u]);
        else {
#pragma unroll
          for (int e = 0; e < 8; e++) v[u][e] = 0.0f;
        }
      }
#pragma unroll
      for (int e = 0; e < 8; e++)
        s[e] += ((v[0][e] + v[1][e]) + (v[2][e] + v[3][e])) + ((v[4][e] + v[5][e]) + (v[6][e] + v[7][e]));
    }
  }
  if (y != 0) {
#pragma unroll
    for (int e = 0; e < 8; e++) red[y - 1][x][e] = s[e];
  }
  __syncthreads();
  if (y != 0 || idx >= hll) return;
#pragma unroll
  for (int k = 0; k < 3; k++)
#pragma unroll
    for (int e = 0; e < 8; e++) s[e] += red[k][x][e];
  st8<float>(dbias + idx, s);
}

// dbiasT[h][j][i] = sum_b dS[b][h][j][i]  (elementwise over the trailing [H][L][L] block)
// 256 threads = 64 groups of 4 consecutive outputs x 4 batch lanes; 8- / 16-byte loads
template <typename T>
__global__ __launch_bounds__(256) void attn_dbias_reduce_kernel(const T* dS, float* dbias, int B, long long hll) {
  __shared__ float red[256][4];
  const int x = threadIdx.x & 63, y = threadIdx.x >> 6;
  const long long idx = ((long long)blockIdx.x * 64 + x) * 4;
  float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (idx < hll) {
    if ((hll & 3) == 0) {
      for (int b = y; b < B; b += 16) {      // 4 independent loads in flight
        float v[4][4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
          int bb = b + 4 * u;
          if (bb < B) load4<T>(dS + (long long)bb * hll + idx, v[u]);
          else { v[u][0] = v[u][1] = v[u][2] = v[u][3] = 0.0f; }
        }
#pragma unroll
        for (int e = 0; e < 4; e++) s[e] += (v[0][e] + v[1][e]) + (v[2][e] + v[3][e]);
      }
    } else {
      for (int b = y; b < B; b += 4)
        for (int e = 0; e < 4; e++)
          if (idx + e < hll) s[e] += to_f(dS[(long long)b * hll + idx + e]);
    }
  }
  red[threadIdx.x][0] = s[0]; red[threadIdx.x][1] = s[1]; red[threadIdx.x][2] = s[2]; red[threadIdx.x][3] = s[3];
  __syncthreads();
  if (y != 0 || idx >= hll) return;
  for (int k = 1; k < 4; k++)
    for (int e = 0; e < 4; e++) s[e] += red[k * 64 + x][e];
  for (int e = 0; e < 4; e++)
    if (idx + e < hll) dbias[idx + e] = s[e];
}
