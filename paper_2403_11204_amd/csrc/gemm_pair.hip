// Weight gradient and optimiser step of a layer in one kernel: dW = dZ^T A (the "NT" product of gemm.hip), then
// v = mu v + dW; w -= lr v on the float32 masters and their copies (paper Sec. 3).  A launch takes up to two products that do not
// depend on each other -- two weight gradients, or one with the data gradient of the layer below -- the layers' biases and the sum
// of the step's loss.
//
// What bounds it is memory: 20 bytes a weight (24 with the gradient stored) where a product and an update behind it move 28, and
// the products hide behind that as far as the two kinds of work overlap.
//   * Two workgroups of 128x128 tiles per compute unit (64 KB of LDS and up to 256 registers each), or three of 64x128 where the
//     launch has no more 128x128 tiles than the chip holds at once: one's streams beside another's multiplies.  64x128 / 128x128,
//     a pass: 784-1500-3001-777 bf16, 1000 rows 547 / 570 us, 784-4096-4096-2048 (1000 to 1300 tiles a launch) 1449 / 1381.
//   * A data gradient in the same launch brings multiplies where the update has none: 1024x4096x4096 and the 2048x4096 update
//     beside it 73 us, one after the other 41 + 23 + 33 with the update apart.
//   * The tile goes through LDS and every stream through memory in whole row segments (512 bytes of the float32 streams, 256 of
//     the bf16 copies); the first half of the weights and momenta is requested before the last k-tile's products, the second
//     behind the accumulators' way into LDS.  Alone, nothing in the caches: with 64-byte segments straight from the accumulators (the epilogue
//     of gemm.hip) on 128x128 tiles 4096x4096x1024 bf16 took 160 us, now 86; product and update apart 104.  2048x2048x512 36, 21, 32;
//     16384x16384x1024 2493, 1167, 1949; float32 2048x2048x256 45, 31, 43.  With K = 64, next to nothing to multiply, 4096x4096 takes 70 us:
//     4.8 TB/s.  In a step of a segment 4096-4096, 1024 rows: 83 us, 94 with the gradient stored as well, apart 41 + 58, on 256x256 tiles with the
//     update in the epilogue of gemm.hip 96 + 5 for the bias.
//   * Weights, momenta and gradients pass the caches by where a step's data do not fit into them (see the caller).
// The order of every sum is that of gemm.hip's tiles and of the 64x64 ones (float32: the same bits).
#include <stddef.h>

#include "elementwise_device.h"
#include "gemm_device.h"

namespace slp {
namespace {

constexpr int kTile = 128;                             // columns of a tile
constexpr int lds_bytes(int bm) { return 2 * (bm + kTile) * 128; }     // two stages; the tile in float32 takes no more
constexpr int kBiasRows = 16;                                                           // output features of one bias workgroup

struct PairLaunch {
  GemmArgs g[2];
  int epi[2], tiles[2], first[2];     // first workgroup of each product, a multiple of 8
  BiasJob bias[2];
  int bias_first[2], sum_first;
  SumJob sum;
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
#define SLP_FENCE() __builtin_amdgcn_sched_barrier(0)
#define SLP_LDS_BARRIER()                            \
  do {                                               \
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); \
    __builtin_amdgcn_s_barrier();                    \
    asm volatile("" ::: "memory");                   \
  } while (0)

// The BM x 128 tile of a product into LDS as float32, row-major: 16-byte chunk c of row r at chunk c ^ (r & 15) (no bank
// conflicts on either side).  request() issues the REQUESTS loads of what the epilogue needs first, behind the last operand loads.
// The caller's next step is a barrier.
template <typename T, int BM, int REQUESTS, typename F>
__device__ __forceinline__ void tile_product(const GemmArgs& g, int m0, int n0, unsigned char* smem, F request) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int ES = sizeof(T), CH = Chunk<T>::elems, BK = 128 / ES;
  typedef Mma<T> MM;
  constexpr int MB = MM::MB, AH = MM::AH, CPS = 64 / MB, KSUB = 8 / CPS, UNITS = KSUB * AH;
  constexpr int kStageBytes = (BM + kTile) * 128;
  constexpr int WTM = BM / 2, WT = kTile / 2, MI = WTM / MB, NI = WT / MB, MIH = MI / AH;      // a wavefront owns BM/2 x 64 of the tile
  constexpr int LA = BM / 32, LB = kTile / 32;             // 16-byte loads per thread, operand and k-tile
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = w & 1, wn = w >> 1, lgrp = lane / MB, lrow = lane % MB;

  const int Kr = (g.K + CH - 1) / CH * CH, nk = (Kr + BK - 1) / BK;
  const __amdgpu_buffer_rsrc_t rsrcA =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.A), 0, (int)((size_t)g.M * g.lda * ES), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcB =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.B), 0, (int)((size_t)g.N * g.ldb * ES), 0x00020000);
  const int prow = w * 8 + (lane >> 3), pc = (lane & 7) ^ ((prow >> 1) & 7);
  const uint32_t a0 = (uint32_t)(((size_t)(m0 + prow) * g.lda + pc * CH) * ES), b0 = (uint32_t)(((size_t)(n0 + prow) * g.ldb + pc * CH) * ES);
  const uint32_t sa = (uint32_t)(32 * g.lda * ES), sb = (uint32_t)(32 * g.ldb * ES);
  auto gload = [&](int kt, int stage, int i) {
    const bool in_k = kt * BK + pc * CH < Kr;      // past the end of K every load becomes a zero fill
    const uint32_t k = (uint32_t)kt * 128u;
    unsigned char* d = smem + stage * kStageBytes + w * 1024;
    if (i < LA) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcA, (lds_ptr_t)(d + i * 4096), 16, in_k ? a0 + i * sa + k : kOutOfRange, 0, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB, (lds_ptr_t)(d + BM * 128 + (i - LA) * 4096), 16,
                                                  in_k ? b0 + (i - LA) * sb + k : kOutOfRange, 0, 0, 0);
  };

  const uint32_t fragA = (uint32_t)((wm * WTM + lrow) * 128), fragB = (uint32_t)(BM * 128 + (wn * WT + lrow) * 128);
  uint32_t xo[KSUB];
#pragma unroll
  for (int kk = 0; kk < KSUB; ++kk) xo[kk] = (uint32_t)(((kk * CPS + lgrp) ^ ((lane >> 1) & 7)) << 4);
  typename MM::acc_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < MM::ACC; ++r) acc[i][j][r] = 0.0f;
  u32x4 af[2][MIH], bfr[2][NI];
  constexpr int NRD = MIH + NI, NLD = LA + LB, NMM = MIH * NI;
  auto reads_of = [](int u) { return MIH + (u % AH == 0 ? NI : 0); };
  auto read_one = [&](int stage, int u, int r) {
    const unsigned char* s = smem + stage * kStageBytes;
    const int kk = u / AH, h = u % AH;
    if (r < MIH) af[u & 1][r] = *(const u32x4*)(s + fragA + (h * MIH + r) * MB * 128 + xo[kk]);
    else bfr[kk & 1][r - MIH] = *(const u32x4*)(s + fragB + (r - MIH) * MB * 128 + xo[kk]);
  };
  // the operands exchanged: a lane's accumulator quad is 4 consecutive columns of one output row, one 16-byte store into LDS
  auto mma_one = [&](int u, int m) {
    MM::mma(acc[(u % AH) * MIH + m / NI][m % NI], bfr[(u / AH) & 1][m % NI], af[u & 1][m / NI]);
  };
  auto unit = [&](int u, int stage, int next, bool reads) {
#pragma unroll
    for (int gq = 0; gq < NRD; ++gq) {
      if (reads) {
#pragma unroll
        for (int r = 2 * gq < reads_of(next) ? 2 * gq : reads_of(next); r < (2 * gq + 2 < reads_of(next) ? 2 * gq + 2 : reads_of(next)); ++r)
          read_one(stage, next, r);
      }
#pragma unroll
      for (int m = gq * NMM / NRD; m < (gq + 1) * NMM / NRD; ++m) mma_one(u, m);
      SLP_FENCE();
    }
  };
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int i = 0; i < NLD; ++i) gload(st, st, i);
  __builtin_amdgcn_s_waitcnt(SLP_VMCNT(NLD));
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NRD; ++r) read_one(0, 0, r);
  for (int kt = 0; kt + 1 < nk; ++kt) {
    const int cur = kt & 1, nxt = cur ^ 1;
#pragma unroll
    for (int u = 0; u < UNITS - 1; ++u) unit(u, cur, u + 1, true);
    __builtin_amdgcn_s_waitcnt(SLP_VMCNT(0));
    __syncthreads();
#pragma unroll
    for (int gq = 0; gq < NRD; ++gq) {
#pragma unroll
      for (int r = 2 * gq < NRD ? 2 * gq : NRD; r < (2 * gq + 2 < NRD ? 2 * gq + 2 : NRD); ++r) read_one(nxt, 0, r);
#pragma unroll
      for (int i = gq * NLD / NRD; i < (gq + 1) * NLD / NRD; ++i) gload(kt + 2, cur, i);
#pragma unroll
      for (int m = gq * NMM / NRD; m < (gq + 1) * NMM / NRD; ++m) mma_one(UNITS - 1, m);
      SLP_FENCE();
    }
  }
  request();
  SLP_FENCE();
  {
    const int cur = (nk - 1) & 1;
#pragma unroll
    for (int u = 0; u < UNITS; ++u) unit(u, cur, u + 1 < UNITS ? u + 1 : u, u + 1 < UNITS);
  }
  __builtin_amdgcn_s_waitcnt(SLP_VMCNT(REQUESTS));      // the zero fills of the last k-tiles are older than the requests
  SLP_LDS_BARRIER();
  constexpr int NQ = MM::ACC / 4;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int p = 0; p < NQ; ++p) {
        const int r = wm * WTM + i * MB + lrow, c = wn * (WT / 4) + j * (MB / 4) + (MB == 32 ? 2 * p : 0) + lgrp;
        *(f32x4*)(smem + r * 512 + ((c ^ (r & 15)) << 4)) = f32x4{acc[i][j][4 * p], acc[i][j][4 * p + 1], acc[i][j][4 * p + 2], acc[i][j][4 * p + 3]};
      }
#endif
}

// From there a thread owns 4 consecutive rows x 4 columns in each strip of 32 rows.
__device__ __forceinline__ f32x4 tile_row(const unsigned char* smem, int s, int e) {
  const int q = threadIdx.x & 31, r = 32 * s + 4 * (threadIdx.x >> 5) + e;
  return *(const f32x4*)(smem + r * 512 + ((q ^ (r & 15)) << 4));
}

// The transposed copy through LDS: the vector of rows 4 p .. 4 p + 3 of column c at place p ^ (c / 4).  turned[strip][column].
template <typename T, int BM>
__device__ __forceinline__ void store_turned(const typename Vec4<T>::type (&turned)[BM / 32][4], void* out, int ld, int M, int N, int m0, int n0,
                                             unsigned char* smem) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int ES = sizeof(T), CH = Chunk<T>::elems;
  const int t = threadIdx.x, q = t & 31, g8 = t >> 5, Mr = (M + 7) & ~7;
  __syncthreads();
#pragma unroll
  for (int s = 0; s < BM / 32; ++s)
#pragma unroll
    for (int c = 0; c < 4; ++c) *(typename Vec4<T>::type*)(smem + (4 * q + c) * (BM * ES) + ((8 * s + g8) ^ (q & (BM / 4 - 1))) * (4 * ES)) = turned[s][c];
  __syncthreads();
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)((size_t)N * ld * ES), 0x00020000);
  constexpr int CPR = BM / CH;         // 16-byte pieces of a column
#pragma unroll
  for (int it = 0; it < kTile * CPR / 256; ++it) {
    const int c = it * (256 / CPR) + t / CPR, k = t % CPR, x = (c >> 2) & (BM / 4 - 1);
    u32x4 v = *(const u32x4*)(smem + c * (BM * ES) + ((k ^ (ES == 2 ? x >> 1 : x)) << 4));
    if (ES == 2 && (x & 1)) v = u32x4{v[2], v[3], v[0], v[1]};     // (bf16: two vectors a piece, exchanged by the lowest bit)
    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, m0 + k * CH < Mr ? (uint32_t)((n0 + c) * ld + m0 + k * CH) * ES : kOutOfRange, 0, 0);
  }
#endif
}

// STREAM: the cache policy of the weights, momenta and the gradient, 2 (non-temporal) or 0
template <typename T, int BM, int STREAM>
__device__ __forceinline__ void update_tile(const GemmArgs& g, int m0, int n0, unsigned char* smem) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int ES = sizeof(T);
  const int q = threadIdx.x & 31, g8 = threadIdx.x >> 5;
  const uint32_t uo = n0 + 4 * q < g.N ? (uint32_t)((m0 + 4 * g8) * g.ldc + n0 + 4 * q) * 4u : kOutOfRange;     // rows past M are past the end
  const int wbytes = (int)((size_t)g.M * g.ldc * 4);
  // what a launch does without has no bytes: loads return zeros, stores go nowhere, and nothing below branches
  const __amdgpu_buffer_rsrc_t rsrcW = __builtin_amdgcn_make_buffer_rsrc(g.uW, 0, wbytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcV = __builtin_amdgcn_make_buffer_rsrc(g.uV, 0, g.mu != 0.0f ? wbytes : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcG = __builtin_amdgcn_make_buffer_rsrc(g.Cf, 0, g.Cf ? wbytes : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcH = __builtin_amdgcn_make_buffer_rsrc(g.uW16, 0, g.uW16 ? wbytes / 2 : 0, 0x00020000);
  u32x4 wv[BM / 64][8], vv[BM / 64][8];     // requested 64 rows at a time
  auto request = [&](int half) {
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const uint32_t o = uo + (uint32_t)((64 * half + 32 * (x >> 2) + (x & 3)) * g.ldc) * 4u;
      wv[half][x] = __builtin_amdgcn_raw_buffer_load_b128(rsrcW, o, 0, STREAM);
      vv[half][x] = __builtin_amdgcn_raw_buffer_load_b128(rsrcV, o, 0, STREAM);
    }
  };
  tile_product<T, BM, 16>(g, m0, n0, smem, [&] { request(0); });
  SLP_FENCE();
  if constexpr (BM > 64) request(1);
  SLP_FENCE();
  SLP_LDS_BARRIER();
  typename Vec4<T>::type turned[BM / 32][4];
#pragma unroll
  for (int s = 0; s < BM / 32; ++s) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t o = uo + (uint32_t)((32 * s + e) * g.ldc) * 4u;
      f32x4 d = tile_row(smem, s, e);
      // past M and N a zero row of one operand times an infinity of the other is NaN: the pads of every stream and copy stay zero
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (m0 + 32 * s + 4 * g8 + e >= g.M || n0 + 4 * q + c >= g.N) d[c] = 0.0f;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, d), rsrcG, o, 0, STREAM);
      const f32x4 vel = g.mu * __builtin_bit_cast(f32x4, vv[s >> 1][4 * (s & 1) + e]) + d;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, vel), rsrcV, o, 0, STREAM);
      const f32x4 wn = __builtin_bit_cast(f32x4, wv[s >> 1][4 * (s & 1) + e]) - g.lr * vel;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, wn), rsrcW, o, 0, STREAM);
      if (ES == 2) {
        const bf16x4 h = {(bf16)wn[0], (bf16)wn[1], (bf16)wn[2], (bf16)wn[3]};
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, h), rsrcH, o >> 1, 0, 0);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) turned[s][c][e] = (T)wn[c];
    }
  }
  if (g.uWT) store_turned<T, BM>(turned, g.uWT, g.ldwt, g.M, g.N, m0, n0, smem);      // (uniform over the launch)
#endif
}

// The data gradient (EPI_DGRAD with a mask): zero where the stored activation, row-major here, is not positive.
template <typename T, int BM>
__device__ __forceinline__ void gradient_tile(const GemmArgs& g, int m0, int n0, unsigned char* smem) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int ES = sizeof(T);
  typedef typename Vec4<T>::type vec4;
  const int q = threadIdx.x & 31, g8 = threadIdx.x >> 5;
  const bool col_ok = n0 + 4 * q < g.N;
  const uint32_t mo = col_ok ? (uint32_t)((m0 + 4 * g8) * g.ldmask + n0 + 4 * q) * ES : kOutOfRange;
  const uint32_t co = col_ok ? (uint32_t)((m0 + 4 * g8) * g.ldc + n0 + 4 * q) * ES : kOutOfRange;
  const __amdgpu_buffer_rsrc_t rsrcM = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.maskT), 0, (int)((size_t)g.M * g.ldmask * ES), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcC = __builtin_amdgcn_make_buffer_rsrc(g.C, 0, g.C ? (int)((size_t)g.M * g.ldc * ES) : 0, 0x00020000);
  vec4 mask[BM / 32][4];
  tile_product<T, BM, BM / 8>(g, m0, n0, smem, [&] {
#pragma unroll
    for (int x = 0; x < BM / 8; ++x) {
      const uint32_t o = mo + (uint32_t)((32 * (x >> 2) + (x & 3)) * g.ldmask) * ES;
      if constexpr (ES == 2) mask[x >> 2][x & 3] = __builtin_bit_cast(vec4, __builtin_amdgcn_raw_buffer_load_b64(rsrcM, o, 0, 0));
      else mask[x >> 2][x & 3] = __builtin_bit_cast(vec4, __builtin_amdgcn_raw_buffer_load_b128(rsrcM, o, 0, 0));
    }
  });
  SLP_LDS_BARRIER();
  vec4 turned[BM / 32][4];
#pragma unroll
  for (int s = 0; s < BM / 32; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f32x4 d = tile_row(smem, s, e);
      vec4 v;
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = (float)mask[s][e][c] > 0.0f ? (T)d[c] : (T)0.0f;     // (pad columns of the activation are zeros)
      const uint32_t o = co + (uint32_t)((32 * s + e) * g.ldc) * ES;
      if constexpr (ES == 2) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rsrcC, o, 0, 0);
      else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rsrcC, o, 0, 0);
#pragma unroll
      for (int c = 0; c < 4; ++c) turned[s][c][e] = v[c];
    }
  if (g.CT) store_turned<T, BM>(turned, g.CT, g.ldct, g.M, g.N, m0, n0, smem);
#endif
}

static_assert(offsetof(PairLaunch, g) == 0, "the kernel reads its products from the start of its arguments");

template <typename T, int BM, int STREAM>
__global__ __launch_bounds__(256, BM == 64 ? 3 : 2) void pair_kernel(const PairLaunch a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int b = blockIdx.x;
  if (b < a.bias_first[0]) {
    const bool second = b >= a.first[1];
#if defined(__HIP_DEVICE_COMPILE__)
    // read at an offset into the argument segment, not as a choice between two of its parts (which goes through memory)
    const GemmArgs& g = ((const GemmArgs*)(const void*)__builtin_amdgcn_kernarg_segment_ptr())[second ? 1 : 0];
#else
    const GemmArgs& g = a.g[0];
#endif
    const int local = second ? b - a.first[1] : b, total = second ? a.tiles[1] : a.tiles[0];
    if (local >= total) return;        // (padding up to the second product's first workgroup)
    // each XCD takes a contiguous range of tiles, walked down groups of 1024 rows
    const int tilesM = (g.M + BM - 1) / BM, tilesN = (g.N + kTile - 1) / kTile;
    const int xcd = local % kXcds, base = total / kXcds, rem = total % kXcds;
    const int tid = xcd * base + (xcd < rem ? xcd : rem) + local / kXcds;
    constexpr int kGroup = 1024 / BM;
    const int width = kGroup * tilesN, first_m = tid / width * kGroup, gsz = tilesM - first_m < kGroup ? tilesM - first_m : kGroup;
    const int m0 = (first_m + tid % width % gsz) * BM, n0 = tid % width / gsz * kTile;
    if ((second ? a.epi[1] : a.epi[0]) == EPI_DGRAD) gradient_tile<T, BM>(g, m0, n0, smem);
    else update_tile<T, BM, STREAM>(g, m0, n0, smem);
  } else if (b < a.sum_first) {
    const bool second = b >= a.bias_first[1];
    const BiasJob& j = second ? a.bias[1] : a.bias[0];
    const int local = second ? b - a.bias_first[1] : b - a.bias_first[0];
    for (int i = 0; i < kBiasRows / 4; ++i)
      bias_grad_update_block<T>(local * (kBiasRows / 4) + i, (const T*)j.dZT, j.ldt, j.N, j.B, j.db, j.b, j.vb, j.lr, j.mu);
  } else {
    reduce_loss_block((double*)smem, a.sum.partials, a.sum.n, a.sum.scale, a.sum.out0, a.sum.out1);
  }
}

template <typename T, int BM, int STREAM>
hipError_t configure() {
  static std::once_flag once;
  static hipError_t result = hipSuccess;
  std::call_once(once, [] { result = hipFuncSetAttribute((const void*)pair_kernel<T, BM, STREAM>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes(BM)); });
  return result;
}

template <typename T, int BM, int STREAM>
hipError_t launch_tiles(const PairLaunch& a, int grid, hipStream_t s) {
  const hipError_t e = configure<T, BM, STREAM>();
  if (e != hipSuccess) return e;
  pair_kernel<T, BM, STREAM><<<grid, 256, lds_bytes(BM), s>>>(a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch(int bm, bool resident, const PairLaunch& a, int grid, hipStream_t s) {
  if (bm == 64) return resident ? launch_tiles<T, 64, 0>(a, grid, s) : launch_tiles<T, 64, 2>(a, grid, s);
  return resident ? launch_tiles<T, 128, 0>(a, grid, s) : launch_tiles<T, 128, 2>(a, grid, s);
}

template <typename T>
hipError_t configure_type() {
  hipError_t e = configure<T, 64, 0>();
  if (e == hipSuccess) e = configure<T, 64, 2>();
  if (e == hipSuccess) e = configure<T, 128, 0>();
  return e == hipSuccess ? configure<T, 128, 2>() : e;
}

// Workgroups of 128-row tiles that the chip holds at once; a launch that has no more of them is split into 64-row ones.  784-N-N-N,
// microseconds a step with a line of 0 / 256 / 512 / 768 / 1024:
//   bf16      256 rows: N = 2048 97.6 / 97.6 / 94.0 / 93.8 / 93.8, 2816 154 / 154 / 154 / 145 / 145, 3584 199 / 199 / 197 / 199 / 192, 4096 236 / 236 /
//             235 / 236 / 236; 1024 rows: N = 2048 130 / 130 / 134 / 134 / 134, 2304 163 / 163 / 171 / 171 / 173, 3072 250 / 251 / 250 / 245 / 244, 3584
//             303 / 302 / 303 / 304 / 302, 5120 673 / 673 / 673 / 673 / 675
//   float32   256 rows: N = 2304 291 / 291 / 282 / 282 / 282, 3072 427 / 427 / 426 / 404 / 403; 1024 rows: N = 2048 541 / 541 / 511 / 510 / 511, 2560 928
//             / 927 / 925 / 888 / 889, 3584 1465 / 1471 / 1449 / 1472 / 1456, 4096 1727 / 1725 / 1718 / 1720 / 1721
// So the split pays up to some 800 tiles, but for bf16 launches of 256 to 512 of them with long contractions, 3-5 % faster on 128 rows.  784-4096-4096-2048,
// 1024 rows, four steps: 1374 us with 512, 1443 with 800.
constexpr long kSlots = 512;

}  // namespace

hipError_t pair_configure_all() {
  const hipError_t e = configure_type<bf16>();
  return e == hipSuccess ? configure_type<float>() : e;
}

hipError_t launch_pair(int dtype, const SmallGroup& group, hipStream_t s) {
  const int es = dtype == 1 ? 2 : 4;
  auto off = [](const void* p) { return ((uintptr_t)p & 15) != 0; };
  if (group.n < 1 || group.n > 2 || group.n_bias < 0 || group.n_bias > 2 || group.has_copy) return hipErrorInvalidValue;
  PairLaunch a{};
  long tiles128 = 0;
  for (int p = 0; p < group.n; ++p) tiles128 += (long)((group.g[p].M + 127) / 128) * ((group.g[p].N + 127) / 128);
  const int bm = tiles128 <= kSlots ? 64 : 128;
  int next = 0;
  for (int p = 0; p < group.n; ++p) {
    const GemmArgs& g = group.g[p];
    if (g.M <= 0 || g.N <= 0 || g.K <= 0 || !g.A || !g.B || off(g.A) || off(g.B) || g.lda % kLdAlign || g.ldb % kLdAlign) return hipErrorInvalidValue;
    // operands, outputs and copies are addressed with 32-bit byte offsets and a 2 GiB sentinel
    auto large = [&](int rows, int ld, int bytes) { return (size_t)rows * ld * bytes >= 0x80000000ull; };
    if (large(g.M, g.lda, es) || large(g.N, g.ldb, es)) return hipErrorInvalidValue;
    const int Nr = round_up(g.N, 4), Mr = round_up(g.M, kLdAlign);
    if (group.epi[p] == EPI_DGRAD) {
      if ((!g.C && !g.CT) || !g.maskT || off(g.maskT) || g.ldmask % kLdAlign || g.ldmask < Nr || large(g.M, g.ldmask, es))
        return hipErrorInvalidValue;
      if (g.C && (off(g.C) || g.ldc % kLdAlign || g.ldc < Nr || large(g.M, g.ldc, es))) return hipErrorInvalidValue;
      if (g.CT && (off(g.CT) || g.ldct % kLdAlign || g.ldct < Mr || large(g.N, g.ldct, es))) return hipErrorInvalidValue;
    } else if (group.epi[p] == EPI_WGRAD_UPDATE) {
      if (!g.uW || !g.uV || off(g.uW) || off(g.uV) || off(g.uW16) || off(g.uWT) || off(g.Cf) || g.ldc % kLdAlign || g.ldc < Nr || large(g.M, g.ldc, 4))
        return hipErrorInvalidValue;
      if (g.uWT && (g.ldwt % kLdAlign || g.ldwt < Mr || large(g.N, g.ldwt, es))) return hipErrorInvalidValue;
    } else {
      return hipErrorInvalidValue;
    }
    a.g[p] = g;
    a.epi[p] = group.epi[p];
    a.tiles[p] = ((g.M + bm - 1) / bm) * ((g.N + kTile - 1) / kTile);
    a.first[p] = round_up(next, kXcds);
    next = a.first[p] + a.tiles[p];
  }
  if (group.n == 1) a.first[1] = next;
  for (int p = 0; p < 2; ++p) {
    a.bias_first[p] = next;
    if (p < group.n_bias) {
      a.bias[p] = group.bias[p];
      next += (group.bias[p].N + kBiasRows - 1) / kBiasRows;
    }
  }
  a.sum_first = next;
  if (group.has_sum) { a.sum = group.sum; ++next; }
  return dtype == 1 ? launch<bf16>(bm, group.resident, a, next, s) : launch<float>(bm, group.resident, a, next, s);
}

}  // namespace slp
