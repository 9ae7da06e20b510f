// Device helpers shared by the matrix-product kernels (gemm.hip, gemm_small.hip).
#pragma once

#include "slp_kernels.h"

namespace slp {
namespace {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kXcds = 8;
constexpr uint32_t kOutOfRange = 0x80000000u;   // byte offset beyond any operand (sizes are checked < 2 GiB)

template <typename T> struct Chunk;
template <> struct Chunk<bf16> { static constexpr int elems = 8; };
template <> struct Chunk<float> { static constexpr int elems = 4; };

// 32x32 block forms (one 16-byte chunk pair per call), used by the contraction-split kernel for small products
__device__ __forceinline__ void mma_chunk(f32x16& acc, const u32x4& a, const u32x4& b, bf16*) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
__device__ __forceinline__ void mma_chunk(f32x16& acc, const u32x4& a, const u32x4& b, float*) {
  const f32x4 af = __builtin_bit_cast(f32x4, a), bfv = __builtin_bit_cast(f32x4, b);
#pragma unroll
  for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[q], bfv[q], acc, 0, 0, 0);
}

// MFMA geometry per element type.  bf16: v_mfma_f32_16x16x32_bf16 (a 16x16 block over 32 k = 4 chunks per row; the
// block's 4 accumulator registers hold rows 4*(lane/16)..+3 of column lane%16); float32: v_mfma_f32_32x32x2_f32, four
// per chunk pair.  MB = block edge, AH = parts the A fragments of one k-sub-step are read in (pipeline units).
template <typename T> struct Mma;
template <> struct Mma<bf16> {
  static constexpr int MB = 16, AH = 2, ACC = 4;
  typedef f32x4 acc_t;
  static __device__ __forceinline__ void mma(acc_t& acc, const u32x4& a, const u32x4& b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  }
};
template <> struct Mma<float> {
  static constexpr int MB = 32, AH = 1, ACC = 16;
  typedef f32x16 acc_t;
  static __device__ __forceinline__ void mma(acc_t& acc, const u32x4& a, const u32x4& b) {
    const f32x4 af = __builtin_bit_cast(f32x4, a), bfv = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[q], bfv[q], acc, 0, 0, 0);
  }
};

template <typename T> struct Vec4;
template <> struct Vec4<bf16> { typedef bf16x4 type; };
template <> struct Vec4<float> { typedef f32x4 type; };

// 4x4 transpose across the 4 lanes of a quad (lanes 4g..4g+3): on return, lane i holds in v[j] what lane j held
// in v[i].  Two butterfly stages of quad-permute DPP moves; every lane of the quad must be active.
__device__ __forceinline__ float quad_xor(float x, bool by_two) {
  const int xi = __builtin_bit_cast(int, x);
  const int r = by_two ? __builtin_amdgcn_update_dpp(0, xi, 0x4E, 0xF, 0xF, true)      // lanes [2,3,0,1]
                       : __builtin_amdgcn_update_dpp(0, xi, 0xB1, 0xF, 0xF, true);     // lanes [1,0,3,2]
  return __builtin_bit_cast(float, r);
}
__device__ __forceinline__ void quad_transpose(float (&v)[4], int lane) {
  const bool b0 = lane & 1, b1 = lane & 2;
  float r;
  r = quad_xor(b0 ? v[0] : v[1], false); if (b0) v[0] = r; else v[1] = r;
  r = quad_xor(b0 ? v[2] : v[3], false); if (b0) v[2] = r; else v[3] = r;
  r = quad_xor(b1 ? v[0] : v[2], true);  if (b1) v[0] = r; else v[2] = r;
  r = quad_xor(b1 ? v[1] : v[3], true);  if (b1) v[1] = r; else v[3] = r;
}

// s_waitcnt immediate: wait until at most n vector-memory operations are outstanding (other counters untouched)
#define SLP_VMCNT(n) ((((n) & 15) | 0x0F70 | (((n) >> 4) << 14)))

}  // namespace
}  // namespace slp
