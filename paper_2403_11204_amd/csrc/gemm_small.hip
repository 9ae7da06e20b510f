// Matrix products of small layers (fewer 128x128 tiles than the chip has compute units): the same "NT" contraction and
// the same epilogues as gemm.hip, for sizes where a launch is over in a few microseconds and what bounds it is latency,
// not the matrix pipe: the time until the first operands arrive, the waits between k-tiles, and -- before this kernel --
// an epilogue that loaded its bias, mask, weights and momenta quad by quad behind the stores of the quad before (loads and
// stores share one counter, so every such load waited for the stores).
//
//   * Everything the epilogue reads is requested before the first operand and held in registers over the k-loop (at most
//     8 per accumulator quad; a wavefront holds one 32x32 block, so there is room).
//   * TILE 16 and 32: the four wavefronts of a workgroup split the CONTRACTION.  Wavefront w multiplies chunk pair w (32 of the
//     128 bytes) of every k-tile; the four partial accumulators are added through LDS (order 0,1,2,3: deterministic, and
//     float32 sums in one order whatever the tile).  What a chip with few workgroups waits for is the chain of one tile's
//     products on one compute unit, which 16x16 tiles spread over four times the units.  Tried and slower: stages private to a
//     wavefront without barriers (its 32-byte strips quadruple the requests: 1000x300x3000 bf16 20 against 8.4), twice the
//     stages (the same), fragments read one step ahead of their products (the branches cost what it hides).
//   * TILE 64: the wavefronts share 64x64 tiles, 32x32 each, one barrier per k-tile, STAGES k-tiles in flight.
//   * Each XCD takes a contiguous range of tiles (float32 256x1024x1024: 12 instead of 33 MB into the eight L2s).
//   * Operand rows are staged as in gemm.hip (128 bytes per row and k-tile, LDS-direct 16-byte loads, XOR swizzle on the
//     global side, out-of-range rows and k-tail chunks read as zero through the buffer resource's range check).
#include "gemm_device.h"

namespace slp {
namespace {

// What the epilogue of one accumulator quad reads, requested before the k-loop.
template <typename T> struct QuadOperands {
  f32x4 w, v;                          // EPI_WGRAD_UPDATE: master weights and momenta of the 4 columns of this lane's row
  typename Vec4<T>::type mask;         // EPI_DGRAD: stored activations of the 4 rows of this lane's column
};

// A quad is 4 rows mb..mb+3 of column n in a lane, and, after the 4x4 transpose inside the quad of lanes, 4 columns
// nb..nb+3 of one row.
template <typename T, int EPI>
__device__ __forceinline__ void request_quad(const GemmArgs& g, int n, int mb, int lane, QuadOperands<T>& o) {
  const int row = mb + (lane & 3), nb = n - (lane & 3);
  if (EPI == EPI_WGRAD_UPDATE) {
    if (row < g.M && nb < g.N) {
      const size_t idx = (size_t)row * g.ldc + nb;
      o.w = *(const f32x4*)(g.uW + idx);
      if (g.mu != 0.0f) o.v = *(const f32x4*)(g.uV + idx);
    }
  } else if (EPI == EPI_DGRAD && g.maskT && n < g.N && mb < ((g.M + 7) & ~7)) {
    o.mask = *(const typename Vec4<T>::type*)((const T*)g.maskT + (size_t)n * g.ldmask + mb);
  }
}

template <typename T, int EPI>
__device__ __forceinline__ void finish_quad(const GemmArgs& g, int n, int mb, float bias, float (&v)[4], int lane,
                                            const QuadOperands<T>& o) {
  typedef typename Vec4<T>::type vec4;
  const bool col_ok = n < g.N;
  const int row = mb + (lane & 3), nb = n - (lane & 3);
  if (EPI == EPI_WGRAD || EPI == EPI_WGRAD_UPDATE) {
    quad_transpose(v, lane);
    const bool in = row < g.M && nb < g.N;
    const size_t idx = (size_t)row * g.ldc + nb;
    if (EPI == EPI_WGRAD) {
      if (in) *(f32x4*)(g.Cf + idx) = f32x4{v[0], v[1], v[2], v[3]};
      return;
    }
    // v = mu v + g; w -= lr v on 4 consecutive weights of one output row (pad columns hold zeros and stay zero), then back
    // through the transpose: one vector store of 4 output rows of one input column into the transposed copy
    float w[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (in) {
      f32x4 vel = f32x4{v[0], v[1], v[2], v[3]};
      if (g.mu != 0.0f) {
        vel = g.mu * o.v + vel;
        *(f32x4*)(g.uV + idx) = vel;
      }
      const f32x4 wn = o.w - g.lr * vel;
      *(f32x4*)(g.uW + idx) = wn;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = wn[e];
      if (g.uW16) *(bf16x4*)((bf16*)g.uW16 + idx) = bf16x4{(bf16)w[0], (bf16)w[1], (bf16)w[2], (bf16)w[3]};
    }
    if (g.uWT) {
      quad_transpose(w, lane);
      if (col_ok && mb < g.M) *(vec4*)((T*)g.uWT + (size_t)n * g.ldwt + mb) = vec4{(T)w[0], (T)w[1], (T)w[2], (T)w[3]};
    }
    return;
  }
  if (mb >= ((g.M + 7) & ~7)) return;       // the same for the whole quad
  if (EPI == EPI_FWD) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] += bias;
      if (g.relu) v[e] = fmaxf(v[e], 0.0f);
    }
  } else if (g.maskT && col_ok) {   // no mask: the gradient w.r.t. the segment input
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (!((float)o.mask[e] > 0.0f)) v[e] = 0.0f;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (mb + e >= g.M || !col_ok) v[e] = 0.0f;
  if (g.CT && col_ok) *(vec4*)((T*)g.CT + (size_t)n * g.ldct + mb) = vec4{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
  if (g.C) {
    quad_transpose(v, lane);
    if (row < g.M && nb < g.N) *(vec4*)((T*)g.C + (size_t)row * g.ldc + nb) = vec4{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
  }
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// 16x16 block; lane -> row lane % 16, k-group lane / 16; the accumulator holds rows 4 * (lane / 16) .. + 3 of column lane % 16.
// bf16: 4 chunks (64 bytes) per row, one per group.  float32: a chunk pair per row, the even chunk in groups 0 and 2, the odd
// one in 1 and 3.  float32 products add one k after the other, the groups of a product in order, so fed like that the order is
// the order of two 32x32x2 products on the pair (first elements of both chunks, second elements, ...): the tile size does not
// change a bit of the result.
__device__ __forceinline__ void mma16(f32x4& acc, const u32x4& a, const u32x4& b, bool, bf16*) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
__device__ __forceinline__ void mma16(f32x4& acc, const u32x4& a, const u32x4& b, bool odd, float*) {
  const f32x4 af = __builtin_bit_cast(f32x4, a), bfv = __builtin_bit_cast(f32x4, b);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(odd ? af[1] : af[0], odd ? bfv[1] : bfv[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(odd ? af[3] : af[2], odd ? bfv[3] : bfv[2], acc, 0, 0, 0);
}

#define SLP_WAIT_BARRIER(n)                            \
  do {                                                 \
    __builtin_amdgcn_s_waitcnt(SLP_VMCNT(n) & 0xF0FF); \
    asm volatile("" ::: "memory");                     \
    __builtin_amdgcn_s_barrier();                      \
    asm volatile("" ::: "memory");                     \
  } while (0)
template <typename T, int TILE, int STAGES, int EPI>
__device__ __forceinline__ void product_tile(const GemmArgs& g, int tm, int tn, unsigned char* smem) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int ES = sizeof(T), CH = Chunk<T>::elems, BK = 128 / ES;
  constexpr int NQ = TILE == 64 ? 4 : 1;       // accumulator quads a lane finishes
  const int m0 = tm * TILE, n0 = tn * TILE;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int half = lane >> 5, l32 = lane & 31, l16 = lane & 15, g16 = lane >> 4;

  // the quads this lane finishes (TILE 16: wavefront 0's lanes, TILE 32: quad w, TILE 64: quads 0..3, 8 rows apart)
  const int mq = TILE == 16 ? m0 + 4 * g16 : (TILE == 32 ? m0 + 8 * w + 4 * half : m0 + (w & 1) * 32 + 4 * half);
  const int n = TILE == 16 ? n0 + l16 : (TILE == 32 ? n0 + l32 : n0 + (w >> 1) * 32 + l32);
  QuadOperands<T> ops[NQ];
  float bias = 0.0f;
  if (TILE != 16 || w == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) request_quad<T, EPI>(g, n, mq + 8 * q, lane, ops[q]);
    if (EPI == EPI_FWD && n < g.N) bias = g.bias[n];
  }

  const int Kr = (g.K + CH - 1) / CH * CH, nk = (Kr + BK - 1) / BK;
  const __amdgpu_buffer_rsrc_t rsrcA =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.A), 0, (int)((size_t)g.M * g.lda * ES), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcB =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.B), 0, (int)((size_t)g.N * g.ldb * ES), 0x00020000);
  const int lr = lane >> 3, lc = lane & 7;     // a load instruction covers 8 rows: this lane's row, its physical chunk
  typedef __attribute__((ext_vector_type(TILE == 16 ? 4 : 16))) float acc_t;
  constexpr int NR = TILE == 16 ? 4 : 16;
  acc_t acc;
#pragma unroll
  for (int r = 0; r < NR; ++r) acc[r] = 0.0f;

  if constexpr (TILE <= 32) {
    // shared stages: [STAGES][KT k-tiles][A TILE rows, B TILE rows][128 bytes].  A load instruction of the workgroup fills 32
    // rows: at TILE 32 8 rows of A, then 8 of B per wavefront; at TILE 16 wavefronts 0, 1 the rows of A, 2, 3 those of B.
    constexpr int KT = TILE == 32 ? 1 : 2, TSZ = 2 * TILE * 128, STAGE = KT * TSZ, HALF = TILE * 128;
    constexpr int LPT = TILE / 16;             // loads of a wavefront per k-tile
    const bool is_b = TILE == 16 && w >= 2;
    const int prow = TILE == 32 ? w * 8 + lr : (w & 1) * 8 + lr;
    const int pc = lc ^ ((prow >> 1) & 7);
    const uint32_t a0 = (uint32_t)(((size_t)(m0 + prow) * g.lda + pc * CH) * ES), b0 = (uint32_t)(((size_t)(n0 + prow) * g.ldb + pc * CH) * ES);
    auto load = [&](int it, int stage) {       // past the end of K every load becomes a zero fill
#pragma unroll
      for (int j = 0; j < KT; ++j) {
        const int kt = it * KT + j;
        const bool ok = kt * BK + pc * CH < Kr;
        const uint32_t k = (uint32_t)kt * 128u;
        unsigned char* d = smem + stage * STAGE + j * TSZ + w * 1024;
        if constexpr (TILE == 32) {
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcA, (lds_ptr_t)d, 16, ok ? a0 + k : kOutOfRange, 0, 0, 0);
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB, (lds_ptr_t)(d + HALF), 16, ok ? b0 + k : kOutOfRange, 0, 0, 0);
        } else {
          if (is_b) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB, (lds_ptr_t)d, 16, ok ? b0 + k : kOutOfRange, 0, 0, 0);
          else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcA, (lds_ptr_t)d, 16, ok ? a0 + k : kOutOfRange, 0, 0, 0);
        }
      }
    };
    // What this wavefront multiplies of every KT k-tiles.  TILE 32 and float32: chunk pair w, chunks 2w and 2w+1, of each
    // (of a k-tile's 8; one chunk each for the two lane halves, at TILE 16 for groups 0, 2 and 1, 3: see mma16).  TILE 16 in
    // bf16, where one product takes 4 chunks: half w & 1 of k-tile w / 2.
    constexpr bool kHalves = TILE == 16 && ES == 2;
    constexpr int NJ = kHalves ? 1 : KT;
    const int frow = TILE == 32 ? l32 : l16;
    const int fch = TILE == 32 ? 2 * w + half : (kHalves ? 4 * (w & 1) + g16 : 2 * w + (g16 & 1));
    const uint32_t fo = (uint32_t)((kHalves ? (w >> 1) * TSZ : 0) + frow * 128 + ((fch ^ ((frow >> 1) & 7)) << 4));
    const int nit = (nk + KT - 1) / KT;        // k-tiles past the end are zeros: their products change nothing
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) load(s, s);
    for (int it = 0; it < nit; ++it) {
      SLP_WAIT_BARRIER((STAGES - 2) * KT * LPT);       // stage `it` has landed; nobody reads the one before any more
      const unsigned char* d = smem + (it & (STAGES - 1)) * STAGE + fo;
      u32x4 af[NJ], bf[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        af[j] = *(const u32x4*)(d + j * TSZ);
        bf[j] = *(const u32x4*)(d + j * TSZ + HALF);
      }
      load(it + STAGES - 1, (it + STAGES - 1) & (STAGES - 1));
      __builtin_amdgcn_sched_barrier(0);               // all reads and loads go out before the first product
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if constexpr (TILE == 32) mma_chunk(acc, af[j], bf[j], (T*)nullptr);
        else mma16(acc, af[j], bf[j], g16 >= 2, (T*)nullptr);
      }
    }
    __builtin_amdgcn_s_waitcnt(SLP_VMCNT(0));
    __syncthreads();                 // every wavefront is done with its stages: they become the reduction buffer
    float* red = (float*)smem;       // [4 wavefronts][NR registers][64 lanes]
#pragma unroll
    for (int r = 0; r < NR; ++r) red[(w * NR + r) * 64 + lane] = acc[r];
    __syncthreads();
    if (TILE == 16 && w != 0) return;
    const int q0 = TILE == 16 ? 0 : 4 * w;     // TILE 32: wavefront w finishes register quad w
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float sum = red[(q0 + e) * 64 + lane];
#pragma unroll
      for (int p = 1; p < 4; ++p) sum += red[(p * NR + q0 + e) * 64 + lane];
      v[e] = sum;
    }
    finish_quad<T, EPI>(g, n, mq, bias, v, lane, ops[0]);
  } else {
    // shared stages: [STAGES][A 64 rows, B 64 rows][128 bytes]; wavefront w loads rows 8 w + lr and 32 + 8 w + lr of both
    constexpr int STAGE = 128 * 128;
    const int prow = w * 8 + lr;
    const int pc = lc ^ ((prow >> 1) & 7);     // rows 32 apart have the same swizzle
    const uint32_t a0 = (uint32_t)(((size_t)(m0 + prow) * g.lda + pc * CH) * ES), b0 = (uint32_t)(((size_t)(n0 + prow) * g.ldb + pc * CH) * ES);
    const uint32_t sa = (uint32_t)(32 * g.lda * ES), sb = (uint32_t)(32 * g.ldb * ES);
    auto load = [&](int kt, int stage) {
      const bool ok = kt * BK + pc * CH < Kr;  // past the end of K every load becomes a zero fill
      const uint32_t k = (uint32_t)kt * 128u;
      unsigned char* d = smem + stage * STAGE + w * 1024;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcA, (lds_ptr_t)(d + i * 4096), 16, ok ? a0 + i * sa + k : kOutOfRange, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB, (lds_ptr_t)(d + 8192 + i * 4096), 16, ok ? b0 + i * sb + k : kOutOfRange, 0, 0, 0);
    };
    uint32_t fo[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) fo[j] = (uint32_t)(l32 * 128 + (((2 * j + half) ^ ((l32 >> 1) & 7)) << 4));
    const uint32_t fa = (uint32_t)((w & 1) * 4096), fb = (uint32_t)(8192 + (w >> 1) * 4096);
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) load(s, s);
    for (int kt = 0; kt < nk; ++kt) {
      SLP_WAIT_BARRIER((STAGES - 2) * 4);        // tile kt has landed; nobody reads the stage of tile kt - 1 any more
      const unsigned char* d = smem + (kt & (STAGES - 1)) * STAGE;
      u32x4 af[4], bf[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        af[j] = *(const u32x4*)(d + fa + fo[j]);
        bf[j] = *(const u32x4*)(d + fb + fo[j]);
      }
      load(kt + STAGES - 1, (kt + STAGES - 1) & (STAGES - 1));
      __builtin_amdgcn_sched_barrier(0);         // all reads and loads go out before the first product
#pragma unroll
      for (int j = 0; j < 4; ++j) mma_chunk(acc, af[j], bf[j], (T*)nullptr);
    }
    __builtin_amdgcn_s_waitcnt(SLP_VMCNT(0));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = acc[4 * q + e];
      finish_quad<T, EPI>(g, n, mq + 8 * q, bias, v, lane, ops[q]);
    }
  }
#endif
}

template <typename T, int TILE, int STAGES>
__global__ __launch_bounds__(256) void small_product_kernel(const GemmArgs g, const int epi) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // consecutive workgroups go round-robin over the 8 XCDs: each XCD gets a contiguous range of tiles, walked along the shorter
  // side of the output, so that its L2 fetches that side's operand once and an eighth of the other
  const int tilesM = (g.M + TILE - 1) / TILE, tilesN = (g.N + TILE - 1) / TILE, total = tilesM * tilesN;
  const int xcd = blockIdx.x % kXcds, base = total / kXcds, rem = total % kXcds;
  const int tid = xcd * base + (xcd < rem ? xcd : rem) + blockIdx.x / kXcds;
  const bool down = tilesM <= tilesN;
  const int tm = down ? tid % tilesM : tid / tilesN, tn = down ? tid / tilesM : tid % tilesN;
  switch (epi) {       // (uniform over the launch)
    case EPI_FWD: product_tile<T, TILE, STAGES, EPI_FWD>(g, tm, tn, smem); break;
    case EPI_DGRAD: product_tile<T, TILE, STAGES, EPI_DGRAD>(g, tm, tn, smem); break;
    case EPI_WGRAD: product_tile<T, TILE, STAGES, EPI_WGRAD>(g, tm, tn, smem); break;
    default: product_tile<T, TILE, STAGES, EPI_WGRAD_UPDATE>(g, tm, tn, smem); break;
  }
}

constexpr int lds_bytes(int tile, int stages) { return stages * (tile == 64 ? 128 : 64) * 128; }

template <typename T, int TILE, int STAGES>
hipError_t configure() {
  static std::once_flag once;
  static hipError_t result = hipSuccess;
  std::call_once(once, [] {
    result = hipFuncSetAttribute((const void*)small_product_kernel<T, TILE, STAGES>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 lds_bytes(TILE, STAGES));
  });
  return result;
}

template <typename T, int TILE, int STAGES>
hipError_t launch(const GemmArgs& g, int epi, hipStream_t s) {
  hipError_t e = configure<T, TILE, STAGES>();
  if (e != hipSuccess) return e;
  const int tiles = ((g.M + TILE - 1) / TILE) * ((g.N + TILE - 1) / TILE);
  small_product_kernel<T, TILE, STAGES><<<tiles, 256, lds_bytes(TILE, STAGES), s>>>(g, epi);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_t(const GemmArgs& g, int epi, int tile, hipStream_t s) {
  if (tile == 64) return launch<T, 64, 4>(g, epi, s);
  if (tile == 32) return launch<T, 32, 4>(g, epi, s);
  return launch<T, 16, 4>(g, epi, s);
}

}  // namespace

// Tile for a product: 64 from 128 64x64 tiles on (fewer leave half of the compute units idle; also where float32's order of
// summation changes from four partial sums to one, so the line stays); else 16 while there are few of them, 32 otherwise.
// Microseconds per launch behind another, tiles 16 / 32, in brackets the kernels this one replaced (32x32 with the contraction
// split and operands loaded by the quad in the epilogue; 64x64):
//   float32  64x128x784 5.0 / 7.3 (6.8)    80x784x1410 7.2 / 11.1 (10.5)   256x47x1024 5.5 / 8.5 (8.0)     1410x80x784 6.3 / 7.4 (7.0)
//            256x512x1024 7.1 / 8.6 (8.2)  256x1024x1024 10.3 / 8.9 (9.0)  2000x100x784 10.8 / 7.5 (7.3)   500x500x500 6.6 / 5.9 (5.6)
//   bf16     1024x47x4096 5.6 / 8.0 (8.4)  64x784x2048 4.1 / 5.3 (5.5)     400x400x2000 6.6 / 5.5 (5.7)    256x1024x4096 12.0 / 8.3 (12.7)
//   64       float32 1024x1024x256 with update 10.5 (11.1)   bf16 1000x3001x1500 19.2 (20.1)   333x3001x1500 9.9 (10.9)
int small_tile(int dtype, int M, int N) {
  auto tiles = [&](int t) { return (long)((M + t - 1) / t) * ((N + t - 1) / t); };
  if (tiles(16) <= (dtype == 1 ? 400 : 512)) return 16;
  return tiles(64) < 128 ? 32 : 64;
}

hipError_t small_configure_all() {
  hipError_t e = configure<bf16, 16, 4>();
  if (e == hipSuccess) e = configure<bf16, 32, 4>();
  if (e == hipSuccess) e = configure<bf16, 64, 4>();
  if (e == hipSuccess) e = configure<float, 16, 4>();
  if (e == hipSuccess) e = configure<float, 32, 4>();
  if (e == hipSuccess) e = configure<float, 64, 4>();
  return e;
}

hipError_t launch_small_product(int dtype, int epi, const GemmArgs& g, hipStream_t s) {
  const int tile = small_tile(dtype, g.M, g.N);
  return dtype == 1 ? launch_t<bf16>(g, epi, tile, s) : launch_t<float>(g, epi, tile, s);
}

}  // namespace slp
