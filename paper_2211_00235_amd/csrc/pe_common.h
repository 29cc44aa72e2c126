// Device-side basics shared by all kernels: storage types, MFMA policy, small helpers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 bf16;
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));

#define PE_DEV __device__ __forceinline__

// ---------------------------------------------------------------------------
// Storage helpers
// ---------------------------------------------------------------------------
template <typename T> PE_DEV float to_f(T v) { return (float)v; }
template <typename T> PE_DEV T from_f(float v) { return (T)v; }

// 16-byte vector of storage elements
template <typename T> struct Vec16;
template <> struct Vec16<bf16> { static constexpr int N = 8; typedef bf16x8 type; };
template <> struct Vec16<float> { static constexpr int N = 4; typedef f32x4 type; };

// 1 / (1 + 2^(-x log2 e)) with the hardware exponential and reciprocal (about 1 ulp each): four instructions;
// the correctly rounded division alone is a ten-instruction sequence.  2^(+large) = inf gives exactly 0.
PE_DEV float sigmoidf_(float x) { return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x * -1.4426950408889634f)); }

// ---------------------------------------------------------------------------
// MFMA policy.  One 32x32 output tile per wave-instruction.
//   Operand A: lane l holds A[row = l%32][k = (l/32)*KP + 0..KP-1]
//   Operand B: lane l holds B[k = (l/32)*KP + 0..KP-1][col = l%32]
//   Accumulator element a (0..15) of lane l: row = 8*(a/4) + 4*(l/32) + a%4, col = l%32
// bf16 uses v_mfma_f32_32x32x16_bf16 (KP = 8, 16 contraction steps per instruction),
// fp32 uses v_mfma_f32_32x32x2_f32 (KP = 1, 2 steps per instruction).
// ---------------------------------------------------------------------------
template <typename T> struct Mma;
template <> struct Mma<bf16> {
  static constexpr int KP = 8;
  static constexpr int KSTEP = 16;
  typedef bf16x8 frag;
  static PE_DEV void mma(f32x16& acc, frag a, frag b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
  }
  static PE_DEV frag load(const bf16* p) { return *reinterpret_cast<const bf16x8*>(p); }
  static PE_DEV frag zero() { frag f; for (int i = 0; i < 8; i++) f[i] = (bf16)0.0f; return f; }
};
template <> struct Mma<float> {
  static constexpr int KP = 1;
  static constexpr int KSTEP = 2;
  typedef float frag;
  static PE_DEV void mma(f32x16& acc, frag a, frag b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
  }
  static PE_DEV frag load(const float* p) { return *p; }
  static PE_DEV frag zero() { return 0.0f; }
};

// row index inside a 32x32 accumulator tile held by (lane group g = lane/32, element a)
PE_DEV int acc_row(int g, int a) { return 8 * (a >> 2) + 4 * g + (a & 3); }

// 32 x 32 accumulator tile as 8 consecutive accumulator rows per lane: elements 8 j + 0..7 of lane (l32, g) -> rows 16 j + 8 g + 0..7 of
// column l32 (an exchange of quads between the two lane halves)
PE_DEV void rows_unpack(const f32x16& acc, int j, float (&v)[8]) {
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[8 * j + i]), __float_as_uint(acc[8 * j + 4 + i]), false, false);
    v[i] = __uint_as_float(r[0]);
    v[4 + i] = __uint_as_float(r[1]);
  }
}

// A piece: 32 rows x 64 bytes, in a wave's own 2 KB of LDS, between the layout in which memory is read and written in 64-byte
// runs (lane q: chunk q % 4 of rows q / 4 and q / 4 + 16) and the fragment layout (lane (l32, g): chunks g and 2 + g of
// row l32).  A global access in which neighbouring lanes are rows apart costs the address unit one cycle per lane: with the
// fragments loaded and the results stored that way the GEMMs of pe_rows.h were no faster than gemm_kernel.
// The chunk index is XOR-ed with (row / 2) % 4: both access patterns fall on distinct banks.
PE_DEV int piece_slot(int row, int c) { return row * 32 + ((c ^ ((row >> 1) & 3)) << 3); }   // element offset
struct RowsPiece {
  bf16* lds;      // this wave's
  int mem[2];     // slots of the memory layout
  int frag[2];    // slots of the fragment layout
  PE_DEV void init(bf16* p, int lane) {
    lds = p;
    mem[0] = piece_slot(lane >> 2, lane & 3); mem[1] = piece_slot((lane >> 2) + 16, lane & 3);
    frag[0] = piece_slot(lane & 31, lane >> 5); frag[1] = piece_slot(lane & 31, 2 + (lane >> 5));
  }
  // LDS operations of one wave execute in order: only the compiler has to keep the two phases apart
  static PE_DEV void phase() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  PE_DEV void to_frag(const bf16x8 (&m)[2], bf16x8& f0, bf16x8& f1) const {
    phase();
    *reinterpret_cast<bf16x8*>(lds + mem[0]) = m[0];
    *reinterpret_cast<bf16x8*>(lds + mem[1]) = m[1];
    phase();
    f0 = *reinterpret_cast<const bf16x8*>(lds + frag[0]);
    f1 = *reinterpret_cast<const bf16x8*>(lds + frag[1]);
  }
  PE_DEV void to_mem(const bf16x8 (&f)[2], bf16x8& m0, bf16x8& m1) const {
    phase();
    *reinterpret_cast<bf16x8*>(lds + frag[0]) = f[0];
    *reinterpret_cast<bf16x8*>(lds + frag[1]) = f[1];
    phase();
    m0 = *reinterpret_cast<const bf16x8*>(lds + mem[0]);
    m1 = *reinterpret_cast<const bf16x8*>(lds + mem[1]);
  }
};
// 4 consecutive k of one row x from an LDS tile stored [k][x] (ds_read_b64_tr_b16): the 16 lanes of a group pass the addresses of
// 4 rows of k x 4 chunks of 4 x, and lane j receives column x0 + j
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
PE_DEV bf16x4 lds_read_tr(const bf16* p) {
  union { s16x4 s; bf16x4 v; } u;
  u.s = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
  return u.v;
}
// the larger of a lane's value and its partner's (lane ^ 32)
PE_DEV float pair_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

PE_DEV float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
PE_DEV float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Host-side launch check used by all launchers.
#define PE_LAUNCH_CHECK() (hipGetLastError())
