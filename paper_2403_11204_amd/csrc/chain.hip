// The forward pass through consecutive narrow layers (at most 64 inputs and outputs) in one launch (paper Sec. 2: the stored response,
// the joined network).  No row of a batch needs another one, so a workgroup carries a strip of 16 rows through all of them in LDS, where a
// launch per product costs 3 us of an almost empty chip and 2.5 us of the host.  What bounds it is latency: the weights of all layers are
// requested at once (64 KB at most), and a layer is then a few products and three barriers.
// Microseconds a pass in a launch each / in one, replayed back to back and (host-bound) called one after the other: float32 60-60-60-47, 64
// rows 7.8 / 5.8 and 13.1 / 7.5, 64-64-64 5.0 / 4.3 and 10.1 / 7.3, 64-64-64-64 2000 rows 8.2 / 5.7; bf16 64-64-64 5.0 / 3.6 and 10.3 / 7.4.
// Layers of up to 128, whose weights came through stages: 784-128-128-128-47 13.1 / 15.3, and 784-80-60 with its first layer 7.7 / 13.1: a
// strip's contraction over 784 on one compute unit takes longer than a launch of its own.
#include <stddef.h>

#include "gemm_device.h"

namespace slp {
namespace {

constexpr int kStrip = 16;
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// LDS: per layer its weights, KT k-tiles of 64 rows of 128 bytes; the strips of the input and of the activations between the layers, 16
// such rows per k-tile; the partial sums of a product.  16-byte chunk c of a row is at chunk c ^ ((row / 2) & 7), as in gemm.hip.
template <typename T> struct Lds {
  static constexpr int KT = kChainWidth * (int)sizeof(T) / 128, W = KT * kChainWidth * 128, STRIP = KT * kStrip * 128;
  static constexpr int strips = kChainLayers * W, red = strips + kChainLayers * STRIP, bytes = red + 4 * 4 * 1024;
};

// What a lane feeds to the products of a block and k-tile, in the order of sums of gemm_small.hip's 16 and 32 tiles (see mma16 there):
// float32: two elements of its chunk, two apart, for one product each; bf16: its chunk for one product, whose second half belongs to
// a second k-tile, which these layers do not have.
__device__ __forceinline__ void products(f32x4& acc, const unsigned char* a, const unsigned char* b, int g16, float*) {
  const float a0 = *(const float*)(a + (g16 >> 1) * 4), a1 = *(const float*)(a + (g16 >> 1) * 4 + 8);
  const float b0 = *(const float*)(b + (g16 >> 1) * 4), b1 = *(const float*)(b + (g16 >> 1) * 4 + 8);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc, 0, 0, 0);
}
__device__ __forceinline__ void products(f32x4& acc, const unsigned char* a, const unsigned char* b, int g16, bf16*) {
  const u32x4 zero = {0, 0, 0, 0}, x = g16 < 2 ? *(const u32x4*)a : zero, y = g16 < 2 ? *(const u32x4*)b : zero;
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), acc, 0, 0, 0);
}

// Four columns n .. n + 3 of row r of a strip.
template <typename T>
__device__ __forceinline__ typename Vec4<T>::type* strip_quad(unsigned char* strip, int r, int n) {
  const int byte = n * (int)sizeof(T), c = (byte >> 4) & 7;
  return (typename Vec4<T>::type*)(strip + (byte >> 7) * (kStrip * 128) + r * 128 + ((c ^ ((r >> 1) & 7)) << 4) + (byte & 15));
}

template <typename T>
__device__ __forceinline__ void strip_forward(const ChainLaunch& a, int index, unsigned char* smem) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef Lds<T> L;
  typedef typename Vec4<T>::type vec4;
  constexpr int ES = sizeof(T), CH = Chunk<T>::elems, BK = 128 / ES;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, g16 = lane >> 4;
  const int m0 = index * kStrip, M = a.M, last = a.layers - 1;
  // what a lane finishes of every output: rows mb .. mb + 3 of column n, and after the transpose inside the quad of lanes columns
  // nb .. nb + 3 of row `row`
  const int n = 16 * w + l16, rb = 4 * g16, mb = m0 + rb, rl = rb + (lane & 3), row = m0 + rl, nb = n - (lane & 3);
  auto strip = [&](int l) { return smem + L::strips + l * L::STRIP; };       // input of layer l

  // everything this workgroup reads: 8 rows of 128 bytes a load; rows and columns outside a matrix become zeros
  const int prow = w * 8 + (lane >> 3), pc = (lane & 7) ^ ((prow >> 1) & 7);      // (rows 32 apart have the same swizzle)
  {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.X), 0, (int)((size_t)M * a.ldx * ES), 0x00020000);
    if (w < 2)
#pragma unroll
      for (int j = 0; j < L::KT; ++j) {
        const int k = j * BK + pc * CH;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(strip(0) + j * (kStrip * 128) + w * 1024), 16,
                                                 k < a.K0 ? (uint32_t)(((size_t)(m0 + prow) * a.ldx + k) * ES) : kOutOfRange, 0, 0, 0);
      }
  }
  float biases[kChainLayers];
#pragma unroll
  for (int l = 0; l < kChainLayers; ++l) {
    const ChainLayer& y = a.layer[l];
    const int K = l ? a.layer[l ? l - 1 : 0].N : a.K0;
    const bool in = l < a.layers;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(y.W), 0, in ? y.N * y.ldk * ES : 0, 0x00020000);
    if (in)                              // (uniform)
#pragma unroll
      for (int j = 0; j < 2 * L::KT; ++j) {
        const int k = (j >> 1) * BK + pc * CH, r = prow + 32 * (j & 1);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(smem + l * L::W + (j >> 1) * (kChainWidth * 128) + (j & 1) * 4096 + w * 1024), 16,
                                                 k < K ? (uint32_t)((r * y.ldk + k) * ES) : kOutOfRange, 0, 0, 0);
      }
    const __amdgpu_buffer_rsrc_t rsrcb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(y.b), 0, in ? y.N * 4 : 0, 0x00020000);
    biases[l] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrcb, (uint32_t)n * 4u, 0, 0));
  }
  __builtin_amdgcn_s_waitcnt(SLP_VMCNT(0));
  __syncthreads();

  // wavefront w multiplies chunk pair w of every k-tile for all blocks, the four partial sums are added through LDS in the order 0, 1, 2, 3, and
  // it finishes block w
  const uint32_t fo = (uint32_t)(l16 * 128 + (((2 * w + (g16 & 1)) ^ ((l16 >> 1) & 7)) << 4));
  float* red = (float*)(smem + L::red);       // [4 partial sums][4 blocks][4 registers][64 lanes]
  vec4 top;                              // this lane's 4 columns of the last layer's output
#pragma unroll
  for (int l = 0; l < kChainLayers; ++l) {
    if (l > last) break;                 // (uniform)
    const int N = a.layer[l].N;
    const unsigned char *x = strip(l) + fo, *y = smem + l * L::W + fo;
#pragma unroll
    for (int j = 0; j < 4; ++j) {        // (blocks past N: zeros)
      f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kt = 0; kt < L::KT; ++kt) products(acc, x + kt * (kStrip * 128), y + kt * (kChainWidth * 128) + j * 2048, g16, (T*)nullptr);
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((w * 4 + j) * 4 + r) * 64 + lane] = acc[r];
    }
    __syncthreads();
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int at = (w * 4 + e) * 64 + lane;
      v[e] = ((red[at] + red[at + 1024]) + red[at + 2048]) + red[at + 3072];
      v[e] += biases[l];
      if (l < last || a.relu_last) v[e] = fmaxf(v[e], 0.0f);
      if (mb + e >= M || n >= N) v[e] = 0.0f;
    }
    quad_transpose(v, lane);
    top = vec4{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
    if (l < last) *strip_quad<T>(strip(l + 1), rl, nb) = top;
    __syncthreads();
  }
  for (int l = 0; l < a.layers; ++l) {
    const ChainLayer& y = a.layer[l];
    if (y.A && row < M && nb < y.N) *(vec4*)((T*)y.A + (size_t)row * y.lda + nb) = l == last ? top : *strip_quad<T>(strip(l + 1), rl, nb);
  }
  const int NL = a.layer[last].N;
  if (row < M && nb < NL) {
    T* o = (T*)a.out + (size_t)row * NL + nb;
    if ((NL & 3) == 0 && ((uintptr_t)a.out & (4 * sizeof(T) - 1)) == 0) *(vec4*)o = top;
    else
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (nb + e < NL) o[e] = top[e];
  }
  // the copy of the input, from where it is
  if (a.copy && row < M && nb < a.K0) *(vec4*)((T*)a.copy + (size_t)row * a.ldcopy + nb) = *strip_quad<T>(strip(0), rl, nb);
#endif
}

template <typename T>
__global__ __launch_bounds__(256) void chain_kernel(const ChainLaunch a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
#if defined(__HIP_DEVICE_COMPILE__)
  {                                      // one word of every cache line of the arguments, all at once (see gemm_small.hip)
    const uint32_t* k = (const uint32_t*)(const void*)__builtin_amdgcn_kernarg_segment_ptr();
    static_assert(sizeof(ChainLaunch) > 192 && sizeof(ChainLaunch) <= 256, "one word of each of 4 lines");
    asm volatile("" ::"s"(k[0]), "s"(k[16]), "s"(k[32]), "s"(k[48]));
  }
#endif
  strip_forward<T>(a, blockIdx.x, smem);
}

template <typename T>
hipError_t configure() {
  static std::once_flag once;
  static hipError_t result = hipSuccess;
  std::call_once(once, [] { result = hipFuncSetAttribute((const void*)chain_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize, Lds<T>::bytes); });
  return result;
}

}  // namespace

hipError_t chain_configure_all() {
  const hipError_t e = configure<bf16>();
  return e == hipSuccess ? configure<float>() : e;
}

hipError_t launch_chain(int dtype, const ChainLaunch& a, hipStream_t s) {
  const int es = dtype == 1 ? 2 : 4, ch = 16 / es;
  auto off = [](const void* p) { return ((uintptr_t)p & 15) != 0; };
  // rows are read in 16-byte pieces; 32-bit byte offsets and a 2 GiB sentinel
  if (a.layers < 1 || a.layers > kChainLayers || a.M <= 0 || a.K0 <= 0 || a.K0 > kChainWidth || !a.X || !a.out || off(a.X) || a.ldx % ch || a.ldx < round_up(a.K0, ch) ||
      (size_t)a.M * a.ldx * es >= 0x80000000ull)
    return hipErrorInvalidValue;
  for (int l = 0; l < a.layers; ++l) {
    const ChainLayer& y = a.layer[l];
    if (y.N <= 0 || y.N > kChainWidth || !y.W || !y.b || off(y.W) || y.ldk % kLdAlign || y.ldk < (l ? a.layer[l - 1].N : a.K0) || y.ldk > (1 << 16)) return hipErrorInvalidValue;
    if (off(y.A) || y.lda % kLdAlign || y.lda < round_up(y.N, 4)) return hipErrorInvalidValue;
  }
  if (a.copy && (off(a.copy) || a.ldcopy % kLdAlign || a.ldcopy < round_up(a.K0, 4))) return hipErrorInvalidValue;
  const hipError_t e = dtype == 1 ? configure<bf16>() : configure<float>();
  if (e != hipSuccess) return e;
  const int grid = (a.M + kStrip - 1) / kStrip;
  if (dtype == 1) chain_kernel<bf16><<<grid, 256, Lds<bf16>::bytes, s>>>(a);
  else chain_kernel<float><<<grid, 256, Lds<float>::bytes, s>>>(a);
  return hipGetLastError();
}

}  // namespace slp
