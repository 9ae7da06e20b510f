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
#include <stddef.h>

#include "elementwise_device.h"
#include "gemm_device.h"

namespace slp {
namespace {

// What the epilogue of one accumulator quad reads, requested before the k-loop.
template <typename T> struct QuadOperands {
  f32x4 w, v;                          // EPI_WGRAD_UPDATE: master weights and momenta of the 4 columns of this lane's row
  typename Vec4<T>::type mask;         // EPI_DGRAD: stored activations of the 4 rows of this lane's column
  int id;                              // EPI_FWD_OUT: class id of this lane's row ...
  f32x4 t;                             // ... and its label's, or the given gradient's, 4 columns
};

// A quad is 4 rows mb..mb+3 of column n in a lane, and, after the 4x4 transpose inside the quad of lanes, 4 columns
// nb..nb+3 of one row.
template <typename T, int EPI>
__device__ __forceinline__ void request_quad(const GemmArgs& g, const OutJob& out, int n, int mb, int lane, QuadOperands<T>& o) {
  const int row = mb + (lane & 3), nb = n - (lane & 3);
  if (EPI == EPI_WGRAD_UPDATE) {
    if (g.uW && row < g.M && nb < g.N) {
      const size_t idx = (size_t)row * g.ldc + nb;
      o.w = *(const f32x4*)(g.uW + idx);
      if (g.mu != 0.0f) o.v = *(const f32x4*)(g.uV + idx);
    }
  } else if (EPI == EPI_DGRAD && g.maskT && n < g.N && mb < ((g.M + 7) & ~7)) {
    o.mask = *(const typename Vec4<T>::type*)((const T*)g.maskT + (size_t)n * g.ldmask + mb);
  } else if (EPI == EPI_FWD_OUT && out.table && row < g.M) {
    o.id = out.y[row];
  }
}

// EPI_FWD_OUT, second part, issued behind the first operand loads: the label's columns wait for the class id
template <typename T>
__device__ __forceinline__ void request_target(const GemmArgs& g, const OutJob& out, int n, int mb, int lane, QuadOperands<T>& o) {
  const int row = mb + (lane & 3), nb = n - (lane & 3);
  o.t = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  if (row >= g.M || nb >= g.N) return;
  const bool whole = (g.N & 3) == 0;     // rows of the caller's dense matrices divide into whole quads
  if (out.table) {
    const float* trow = out.table + (size_t)min(max(o.id, 0), out.classes - 1) * g.N + nb;   // ids are the caller's; never index outside the table
    if (whole) o.t = *(const f32x4*)trow;
    else
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (nb + e < g.N) o.t[e] = trow[e];
  } else {
    const T* erow = (const T*)out.ext + (size_t)row * g.N + nb;
    if (whole && ((uintptr_t)out.ext & (4 * sizeof(T) - 1)) == 0) {
      const typename Vec4<T>::type v = *(const typename Vec4<T>::type*)erow;
#pragma unroll
      for (int e = 0; e < 4; ++e) o.t[e] = (float)v[e];
    } else
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (nb + e < g.N) o.t[e] = (float)erow[e];
  }
}

template <typename T, int EPI>
__device__ __forceinline__ void finish_quad(const GemmArgs& g, const OutJob& out, int n, int mb, float bias, float (&v)[4], int lane,
                                            const QuadOperands<T>& o, float& loss) {
  typedef typename Vec4<T>::type vec4;
  const bool col_ok = n < g.N;
  const int row = mb + (lane & 3), nb = n - (lane & 3);
  const bool in = row < g.M && nb < g.N;
  if (EPI == EPI_WGRAD_UPDATE) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (!col_ok) v[e] = 0.0f;              // (an infinity times the zeros past the operand is NaN)
    quad_transpose(v, lane);
    const size_t idx = (size_t)row * g.ldc + nb;
    if (g.Cf && in) *(f32x4*)(g.Cf + idx) = f32x4{v[0], v[1], v[2], v[3]};
    if (!g.uW) return;
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
  if (EPI == EPI_FWD || EPI == EPI_FWD_OUT) {
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
  if (EPI != EPI_FWD_OUT && !g.C && !g.C2) return;
  quad_transpose(v, lane);
  const vec4 r = vec4{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
  if (g.C && in) *(vec4*)((T*)g.C + (size_t)row * g.ldc + nb) = r;
  if (g.C2 && in) {
    T* c2 = (T*)g.C2 + (size_t)row * g.ldc2 + nb;
    if (((g.ldc2 | g.N) & 3) == 0 && ((uintptr_t)g.C2 & (4 * sizeof(T) - 1)) == 0) *(vec4*)c2 = r;
    else
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (nb + e < g.N) c2[e] = r[e];
  }
  if (EPI == EPI_FWD_OUT) {
    float d[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (row < g.M) {
      if (out.table && nb == 0 && (o.id < 0 || o.id >= out.classes)) atomicAdd(out.bad_ids, 1u);   // once per row; rare, and the count is an integer
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (nb + e < g.N) {
          const float a = (float)r[e];
          if (out.table) {
            const float diff = a - o.t[e];
            loss += diff * diff;
            d[e] = out.scale * diff;
          } else d[e] = o.t[e];
          if (g.relu && !(a > 0.0f)) d[e] = 0.0f;
        }
    }
    if (in) *(vec4*)((T*)out.dZ + (size_t)row * out.lddz + nb) = vec4{(T)d[0], (T)d[1], (T)d[2], (T)d[3]};
    quad_transpose(d, lane);
    if (col_ok) *(vec4*)((T*)out.dZT + (size_t)n * out.lddzt + mb) = vec4{(T)d[0], (T)d[1], (T)d[2], (T)d[3]};
  }
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// LDS: four stages of 16 KB at TILE 64, of 8 KB at TILE 16 and 32 (several workgroups per compute unit), and 64 bytes behind
// the 32 or 64 KB for the partial sums of the loss
constexpr int kStages = 4, kTailBytes = 64, kLds32 = kStages * 64 * 128 + kTailBytes, kLds64 = kStages * 128 * 128 + kTailBytes;

// 16x16 block; lane -> row lane % 16, k-group lane / 16; the accumulator holds rows 4 * (lane / 16) .. + 3 of column lane % 16.
// A product adds its groups in order, so what they are fed with keeps the order that the 32x32 block's products have, and the
// choice between tiles 16 and 32 does not change a bit of the result in either type.  bf16: 4 chunks per row, one per group,
// chunk pair w of two successive k-tiles: the order of two 32x32x16 products.  float32: a chunk pair per row, the even chunk in
// groups 0 and 2, the odd one in 1 and 3: the order of two 32x32x2 products on the pair (first elements of both chunks, second
// elements, ...).
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
__device__ __forceinline__ void product_tile(const GemmArgs& g, const OutJob& out, int tm, int tn, int tile_index, unsigned char* smem) {
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
  float bias = 0.0f, loss = 0.0f;
  if (TILE != 16 || w == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) request_quad<T, EPI>(g, out, n, mq + 8 * q, lane, ops[q]);
    if ((EPI == EPI_FWD || EPI == EPI_FWD_OUT) && n < g.N) bias = g.bias[n];
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
    // What this wavefront multiplies of every KT k-tiles: chunk pair w, chunks 2w and 2w+1, of each (of a k-tile's 8; one chunk
    // each for the two lane halves, at TILE 16 for groups 0, 2 and 1, 3: see mma16).  TILE 16 in bf16, where one product takes 4
    // chunks: the pairs of both k-tiles, the first in groups 0 and 1, the second in 2 and 3.
    constexpr bool kBoth = TILE == 16 && ES == 2;
    constexpr int NJ = kBoth ? 1 : KT;
    const int frow = TILE == 32 ? l32 : l16;
    const int fch = TILE == 32 ? 2 * w + half : 2 * w + (g16 & 1);
    const uint32_t fo = (uint32_t)((kBoth ? (g16 >> 1) * TSZ : 0) + frow * 128 + ((fch ^ ((frow >> 1) & 7)) << 4));
    const int nit = (nk + KT - 1) / KT;        // k-tiles past the end are zeros: their products change nothing
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) load(s, s);
    if (EPI == EPI_FWD_OUT && (TILE != 16 || w == 0)) request_target<T>(g, out, n, mq, lane, ops[0]);
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
    finish_quad<T, EPI>(g, out, n, mq, bias, v, lane, ops[0], loss);
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
    if (EPI == EPI_FWD_OUT) {
#pragma unroll
      for (int q = 0; q < 4; ++q) request_target<T>(g, out, n, mq + 8 * q, lane, ops[q]);
    }
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
      finish_quad<T, EPI>(g, out, n, mq + 8 * q, bias, v, lane, ops[q], loss);
    }
  }
  if (EPI == EPI_FWD_OUT && out.table) {     // one partial sum per tile, the wavefronts' added in a fixed order
    loss = wave_sum(loss);
    if (TILE == 16) {
      if (lane == 0) out.partials[tile_index] = loss;
    } else {
      float* part = (float*)(smem + (TILE == 64 ? kLds64 : kLds32) - kTailBytes);
      if (lane == 0) part[w] = loss;
      __syncthreads();
      if (t == 0) out.partials[tile_index] = (part[0] + part[1]) + (part[2] + part[3]);
    }
  }
#endif
}

struct GroupLaunch {
  SmallGroup s;                   // (g[0], g[1] first)
  int tile[2], tiles[2];          // per product: tile edge, number of tiles
  int first[2];                   // first workgroup of each product, a multiple of 8
  int bias_first[2], sum_first, copy_first;
};

// Consecutive workgroups go round-robin over the 8 XCDs: each XCD gets a contiguous range of tiles, walked along the shorter
// side of the output, so that its L2 fetches that side's operand once and an eighth of the other.
template <int TILE>
__device__ __forceinline__ void walk(const GemmArgs& g, uint32_t local, uint32_t total, int& tm, int& tn, int& tid) {
  const uint32_t tilesM = (g.M + TILE - 1) / TILE, tilesN = (g.N + TILE - 1) / TILE;
  const uint32_t xcd = local % kXcds, base = total / kXcds, rem = total % kXcds;
  const uint32_t t = xcd * base + (xcd < rem ? xcd : rem) + local / kXcds;
  const bool down = tilesM <= tilesN;
  const uint32_t shorter = down ? tilesM : tilesN, q = t / shorter, r = t - q * shorter;
  tm = down ? r : q;
  tn = down ? q : r;
  tid = t;
}

template <typename T, int TILE>
__device__ __forceinline__ void product_block(const GemmArgs& g, int epi, const OutJob& out, int local, int total, unsigned char* smem) {
  if (local >= total) return;     // (padding up to the next product's first workgroup)
  int tm, tn, tid;
  walk<TILE>(g, local, total, tm, tn, tid);
  switch (epi) {
    case EPI_FWD: product_tile<T, TILE, kStages, EPI_FWD>(g, out, tm, tn, tid, smem); break;
    case EPI_DGRAD: product_tile<T, TILE, kStages, EPI_DGRAD>(g, out, tm, tn, tid, smem); break;
    case EPI_WGRAD:               // (the same without uW)
    case EPI_WGRAD_UPDATE: product_tile<T, TILE, kStages, EPI_WGRAD_UPDATE>(g, out, tm, tn, tid, smem); break;
    default: product_tile<T, TILE, kStages, EPI_FWD_OUT>(g, out, tm, tn, tid, smem); break;
  }
}

static_assert(offsetof(GroupLaunch, s) == 0 && offsetof(SmallGroup, g) == 0, "the kernel reads its products from the start of its arguments");

// One launch: the tiles of up to two products, then the bias gradients, the sum of the loss and the input's copies, a range of
// workgroups each.  Everything that selects a path is uniform over a workgroup.
template <typename T>
__global__ __launch_bounds__(256) void small_group_kernel(const GroupLaunch a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int b = blockIdx.x;
#if defined(__HIP_DEVICE_COMPILE__)
  // One word of every cache line of the arguments, all at once: the choices below read them in three dependent steps, each of
  // which would wait for memory (0.5 us a launch: 64x64x128 float32 3.8 -> 3.3, 256x1024x1024 9.8 -> 9.3).
  {
    const uint32_t* w = (const uint32_t*)(const void*)__builtin_amdgcn_kernarg_segment_ptr();
    static_assert(sizeof(GroupLaunch) > 704 && sizeof(GroupLaunch) <= 768, "one word of each of 12 lines");
    asm volatile("" ::"s"(w[0]), "s"(w[16]), "s"(w[32]), "s"(w[48]), "s"(w[64]), "s"(w[80]), "s"(w[96]), "s"(w[112]), "s"(w[128]), "s"(w[144]),
                 "s"(w[160]), "s"(w[176]));
  }
#endif
  if (b < a.bias_first[0]) {
    const bool second = a.s.n > 1 && b >= a.first[1];
    // read at an offset into the argument segment, not as a choice between two of its parts (which goes through memory)
#if defined(__HIP_DEVICE_COMPILE__)
    const GemmArgs& g = ((const GemmArgs*)(const void*)__builtin_amdgcn_kernarg_segment_ptr())[second ? 1 : 0];
#else
    const GemmArgs& g = a.s.g[0];
#endif
    const int epi = second ? a.s.epi[1] : a.s.epi[0], tile = second ? a.tile[1] : a.tile[0];
    const int total = second ? a.tiles[1] : a.tiles[0], local = second ? b - a.first[1] : b;
    if (tile == 16) product_block<T, 16>(g, epi, a.s.out, local, total, smem);
    else if (tile == 32) product_block<T, 32>(g, epi, a.s.out, local, total, smem);
    else product_block<T, 64>(g, epi, a.s.out, local, total, smem);
  } else if (b < a.sum_first) {
    const bool second = b >= a.bias_first[1];
    const BiasJob& j = second ? a.s.bias[1] : a.s.bias[0];
    bias_grad_update_block<T>(second ? b - a.bias_first[1] : b - a.bias_first[0], (const T*)j.dZT, j.ldt, j.N, j.B, j.db, j.b, j.vb, j.lr, j.mu);
  } else if (b < a.copy_first) {
    reduce_loss_block((double*)smem, a.s.sum.partials, a.s.sum.n, a.s.sum.scale, a.s.sum.out0, a.s.sum.out1);
  } else {
    const CopyJob& c = a.s.copy;
    const int local = b - a.copy_first, across = (c.C + 63) / 64;
    copy_transpose_block<T, 64>(local % across, local / across, (typename Vec16<T>::type*)smem, (const T*)c.in, c.ldin, c.R, c.C,
                                (T*)c.out, c.ldo, (T*)c.outT, c.ldt, c.rows_t, nullptr, 0);
  }
}

// A forward product or a data gradient by itself: a quarter of the arguments and nothing to choose from them.  Microseconds a launch,
// the kernel above / this one (in brackets the kernel that both replaced): float32 1045x192x99 5.1 / 3.4 (3.4), 640x320x632 6.8 /
// 6.2 (6.2), 640x632x26 3.9 / 3.3 (3.6), 64x64x35 3.0 / 2.6 (2.7), 2048x1024x30 8.0 / 6.9 (7.3); bf16 500x500x47 3.2 / 2.7 (2.8).
template <typename T, int TILE, int EPI>
__global__ __launch_bounds__(256) void small_product_kernel(const GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
#if defined(__HIP_DEVICE_COMPILE__)
  {                               // (as above)
    const uint32_t* w = (const uint32_t*)(const void*)__builtin_amdgcn_kernarg_segment_ptr();
    static_assert(sizeof(GemmArgs) > 128 && sizeof(GemmArgs) <= 192, "one word of each of 3 lines");
    asm volatile("" ::"s"(w[0]), "s"(w[16]), "s"(w[32]));
  }
#endif
  int tm, tn, tid;
  walk<TILE>(g, blockIdx.x, ((g.M + TILE - 1) / TILE) * ((g.N + TILE - 1) / TILE), tm, tn, tid);
  const OutJob none{};
  product_tile<T, TILE, kStages, EPI>(g, none, tm, tn, tid, smem);
}

template <typename T, int EPI>
hipError_t launch_product(const GemmArgs& g, int tile, int tiles, hipStream_t s) {
  if (tile == 16) small_product_kernel<T, 16, EPI><<<tiles, 256, kLds32, s>>>(g);
  else if (tile == 32) small_product_kernel<T, 32, EPI><<<tiles, 256, kLds32, s>>>(g);
  else small_product_kernel<T, 64, EPI><<<tiles, 256, kLds64, s>>>(g);
  return hipGetLastError();
}

// The last layer's forward product and the cross-entropy behind it, for up to 64 classes: a workgroup owns 16 rows with all their columns (NT
// tiles of 16), so that their logits need not be in memory before the loss is formed from them.  The products are those of TILE 16 above,
// column tile by column tile, the rows' arithmetic that of the cross-entropy kernel: the same bits.  What bounds it is one
// compute unit's stream of 16 rows of activations and all rows of the weights, where the product by itself spreads the columns over NT units;
// six stages keep 80 KB of it in flight.  See logits_fit for where it is used.
constexpr int kLogitStages = 6;
constexpr int logit_lds(int nt) { return kLogitStages * 2 * 16 * (1 + nt) * 128; }
template <typename T, int NT>
__global__ __launch_bounds__(256) void logits_xent_kernel(const GemmArgs g, const OutJob out) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int ES = sizeof(T), CH = Chunk<T>::elems, BK = 128 / ES;
  constexpr int ROWS = 16 * (1 + NT), TSZ = ROWS * 128, STAGE = 2 * TSZ, NLD = 1 + NT;      // a stage: two k-tiles; loads of a wavefront per stage
  constexpr bool kBoth = ES == 2;
  constexpr int NJ = kBoth ? 1 : 2;
  const int m0 = blockIdx.x * 16;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l16 = lane & 15, g16 = lane >> 4;
  // what the end needs, ahead of the operands: the bias of this wavefront's column tile, the class ids of its four rows
  const int n = w * 16 + l16, mr = m0 + 4 * w;
  const float bias = w < NT && n < g.N ? g.bias[n] : 0.0f;
  int cls[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) cls[r] = out.y[min(mr + r, g.M - 1)];

  const int Kr = (g.K + CH - 1) / CH * CH, nk = (Kr + BK - 1) / BK, nit = (nk + 1) / 2;
  const __amdgpu_buffer_rsrc_t rsrcA =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.A), 0, (int)((size_t)g.M * g.lda * ES), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcB =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.B), 0, (int)((size_t)g.N * g.ldb * ES), 0x00020000);
  // load i of wavefront w is number q = w + 4 i of a stage's: rows 8 (q mod ROWS / 8) .. + 7 of its k-tile q / (ROWS / 8)
  const int lr = lane >> 3, lc = lane & 7;
  uint32_t off[NLD];
  int chunk[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int q = w + 4 * i, j = q / (ROWS / 8), row = q % (ROWS / 8) * 8 + lr;
    const int pc = lc ^ (((row & 15) >> 1) & 7);
    chunk[i] = j * BK + pc * CH;
    off[i] = (uint32_t)((row < 16 ? (size_t)(m0 + row) * g.lda : (size_t)(row - 16) * g.ldb) * ES) + (uint32_t)chunk[i] * ES;
  }
  auto load = [&](int it, int stage) {         // past the end of K every load becomes a zero fill
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int q = w + 4 * i;
      const uint32_t o = it * 2 * BK + chunk[i] < Kr ? off[i] + (uint32_t)it * 256u : kOutOfRange;
      const lds_ptr_t d = (lds_ptr_t)(smem + stage * STAGE + q * 1024);
      if (q % (ROWS / 8) < 2) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcA, d, 16, o, 0, 0, 0);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB, d, 16, o, 0, 0, 0);
    }
  };
  const uint32_t fo = (uint32_t)((kBoth ? (g16 >> 1) * TSZ : 0) + l16 * 128 + (((2 * w + (g16 & 1)) ^ ((l16 >> 1) & 7)) << 4));
  f32x4 acc[NT];
#pragma unroll
  for (int c = 0; c < NT; ++c) acc[c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < kLogitStages - 1; ++s) load(s, s);
  int stage = 0, next = kLogitStages - 1;
  for (int it = 0; it < nit; ++it) {
    SLP_WAIT_BARRIER((kLogitStages - 2) * NLD);        // stage `it` has landed; nobody reads the one before any more
    const unsigned char* d = smem + stage * STAGE + fo;
    u32x4 af[NJ], bf[NJ][NT];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      af[j] = *(const u32x4*)(d + j * TSZ);
#pragma unroll
      for (int c = 0; c < NT; ++c) bf[j][c] = *(const u32x4*)(d + j * TSZ + (1 + c) * 2048);
    }
    load(it + kLogitStages - 1, next);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int c = 0; c < NT; ++c) mma16(acc[c], af[j], bf[j][c], g16 >= 2, (T*)nullptr);
    stage = stage + 1 == kLogitStages ? 0 : stage + 1;
    next = next + 1 == kLogitStages ? 0 : next + 1;
  }
  __builtin_amdgcn_s_waitcnt(SLP_VMCNT(0));
  __syncthreads();                 // the stages become the reduction buffer, [4 wavefronts][NT tiles][4 registers][64 lanes] ...
  float* red = (float*)smem;
  float* logits = red + 4 * NT * 256;        // ... and behind it the logits, [16 rows][64 columns]
#pragma unroll
  for (int c = 0; c < NT; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) red[((w * NT + c) * 4 + e) * 64 + lane] = acc[c][e];
  __syncthreads();
  if (w < NT) {                    // wavefront w finishes column tile w: rows 4 g16 .. + 3 of column n
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = red[(w * 4 + e) * 64 + lane];
#pragma unroll
      for (int p = 1; p < 4; ++p) v += red[((p * NT + w) * 4 + e) * 64 + lane];
      v += bias;
      if (g.relu) v = fmaxf(v, 0.0f);
      logits[(4 * g16 + e) * 64 + n] = (float)(T)v;
    }
  }
  __syncthreads();
  if (mr >= ((g.M + 7) & ~7)) return;
  float zv[1][4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = min(4 * w + r, g.M - 1 - m0);          // rows past the batch take its last one and store zeros
    zv[0][r] = lane < g.N ? logits[row * 64 + lane] : -INFINITY;
    if (mr + r < g.M && lane < g.N) ((T*)g.C)[(size_t)(mr + r) * g.ldc + lane] = (T)zv[0][r];
  }
  xent_rows<T, 1>(zv, cls, [&](int r, int id) { return logits[min(4 * w + r, g.M - 1 - m0) * 64 + id]; }, mr, g.M, g.N, g.relu, out.scale, (T*)out.dZ,
                  out.lddz, (T*)out.dZT, out.lddzt, out.partials, out.bad_ids);
#endif
}

template <typename T, int NT>
hipError_t configure_logits() {
  static std::once_flag once;
  static hipError_t result = hipSuccess;
  std::call_once(once, [] { result = hipFuncSetAttribute((const void*)logits_xent_kernel<T, NT>, hipFuncAttributeMaxDynamicSharedMemorySize, logit_lds(NT)); });
  return result;
}
template <typename T, int NT>
hipError_t launch_logits_nt(const GemmArgs& g, const OutJob& out, hipStream_t s) {
  const hipError_t e = configure_logits<T, NT>();
  if (e != hipSuccess) return e;
  logits_xent_kernel<T, NT><<<(((g.M + 7) & ~7) + 15) / 16, 256, logit_lds(NT), s>>>(g, out);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_logits_t(const GemmArgs& g, const OutJob& out, hipStream_t s) {
  switch ((g.N + 15) / 16) {
    case 1: return launch_logits_nt<T, 1>(g, out, s);
    case 2: return launch_logits_nt<T, 2>(g, out, s);
    case 3: return launch_logits_nt<T, 3>(g, out, s);
    case 4: return launch_logits_nt<T, 4>(g, out, s);
    default: return hipErrorInvalidValue;
  }
}
template <typename T>
hipError_t configure_logits_all() {
  hipError_t e = configure_logits<T, 1>();
  if (e == hipSuccess) e = configure_logits<T, 2>();
  if (e == hipSuccess) e = configure_logits<T, 3>();
  return e == hipSuccess ? configure_logits<T, 4>() : e;
}

template <typename T>
hipError_t configure() {
  static std::once_flag once;
  static hipError_t result = hipSuccess;
  std::call_once(once, [] {
    const void* kernels[] = {(const void*)small_group_kernel<T>, (const void*)small_product_kernel<T, 64, EPI_FWD>,
                             (const void*)small_product_kernel<T, 64, EPI_DGRAD>};
    for (const void* k : kernels)
      if (result == hipSuccess) result = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLds64);
  });
  return result;
}

}  // namespace

// Tile for a product: 64 from 128 64x64 tiles on (fewer leave half of the compute units idle; also where the order of
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

int small_tile_count(int dtype, int M, int N) {
  const int t = small_tile(dtype, M, N);
  return ((M + t - 1) / t) * ((N + t - 1) / t);
}

hipError_t small_configure_all() {
  hipError_t e = configure<bf16>();
  if (e == hipSuccess) e = configure<float>();
  if (e == hipSuccess) e = configure_logits_all<bf16>();
  return e == hipSuccess ? configure_logits_all<float>() : e;
}

// One launch less against columns that share a compute unit, whose float32 matrix rate is then the limit.  A step of 64-K-C on the device alone, rows
// 1 / 64 / 1000, microseconds, product and cross-entropy apart -> in one launch:
//   float32 1536-16 18.9 / 21.4 / 36.2 -> 18.0 / 19.8 / 34.2, 512-32 15.7 / 17.2 / 26.3 -> 15.3 / 16.1 / 26.2, 768-32 16.4 / 17.8 / 29.5 -> 16.4 / 17.6 /
//   30.0, 256-48 15.0 / 16.1 / 21.4 -> 14.5 / 15.8 / 21.3, 384-48 15.4 / 16.8 / 23.4 -> 15.7 / 16.7 / 24.0, 128-64 14.7 / 15.8 / 20.7 -> 14.4 / 15.5 /
//   20.2, 256-64 15.2 / 16.2 / 21.7 -> 15.4 / 16.6 / 22.3;
//   bf16 4096-16 20.2 / 22.8 / 39.7 -> 18.8 / 20.4 / 36.6, 4096-47 22.0 / 24.4 / 41.0 -> 22.1 / 23.7 / 40.4, 6144-47 26.6 / 29.6 / 53.1 -> 27.5 / 29.8 /
//   52.2, 1024-64 15.8 / 17.7 / 23.4 -> 15.7 / 16.8 / 22.3, 2048-64 17.3 / 19.6 / 31.5 -> 17.7 / 19.2 / 31.1, 4096-64 22.2 / 24.6 / 41.5 -> 23.2 / 25.1 /
//   41.8.
bool logits_fit(int dtype, int M, int N, int K) {
  if (N > 64 || !product_is_small(dtype, EPI_FWD, M, N) || small_tile(dtype, M, N) != 16) return false;
  const int nt = (N + 15) / 16;
  return dtype == 1 ? K <= (nt == 4 ? 1024 : 4096) : K <= 1536 && nt * nt * K <= 2304;
}

hipError_t launch_logits(int dtype, const GemmArgs& g, const OutJob& out, hipStream_t s) {
  const int es = dtype == 1 ? 2 : 4, ch = 16 / es;
  auto off = [](const void* p) { return ((uintptr_t)p & 15) != 0; };
  if (g.M <= 0 || g.N <= 0 || g.N > 64 || g.K <= 0 || !g.A || !g.B || off(g.A) || off(g.B) || g.lda % ch || g.ldb % ch) return hipErrorInvalidValue;
  if ((size_t)g.M * g.lda * es >= 0x80000000ull || (size_t)g.N * g.ldb * es >= 0x80000000ull) return hipErrorInvalidValue;
  if (!g.bias || !g.C || g.ldc < g.N || !out.y || !out.partials || !out.bad_ids || !out.dZ || out.lddz < g.N) return hipErrorInvalidValue;
  if (out.dZT && (off(out.dZT) || out.lddzt % kLdAlign)) return hipErrorInvalidValue;
  return dtype == 1 ? launch_logits_t<bf16>(g, out, s) : launch_logits_t<float>(g, out, s);
}

hipError_t launch_small_group(int dtype, const SmallGroup& group, hipStream_t s) {
  const int es = dtype == 1 ? 2 : 4, ch = 16 / es;
  auto off = [](const void* p) { return ((uintptr_t)p & 15) != 0; };
  if (group.n < 1 || group.n > 2 || group.n_bias < 0 || group.n_bias > 2) return hipErrorInvalidValue;
  GroupLaunch a{};
  a.s = group;
  int next = 0, lds = kLds32;
  for (int p = 0; p < group.n; ++p) {
    if (group.epi[p] == EPI_WGRAD) a.s.g[p].uW = nullptr;      // the kernel's mark for a gradient without an update
    const GemmArgs& g = group.g[p];
    const int epi = group.epi[p];
    if (g.M <= 0 || g.N <= 0 || g.K <= 0 || !g.A || !g.B || off(g.A) || off(g.B) || g.lda % ch || g.ldb % ch) return hipErrorInvalidValue;
    // operands are addressed with 32-bit byte offsets and a 2 GiB sentinel
    if ((size_t)g.M * g.lda * es >= 0x80000000ull || (size_t)g.N * g.ldb * es >= 0x80000000ull) return hipErrorInvalidValue;
    if (epi == EPI_WGRAD || epi == EPI_WGRAD_UPDATE) {
      if (g.ldc % 4 || off(g.Cf) || (epi == EPI_WGRAD && !g.Cf)) return hipErrorInvalidValue;
      if (epi == EPI_WGRAD_UPDATE && (!g.uW || !g.uV || off(g.uW) || off(g.uV) || off(g.uW16) || off(g.uWT) || (g.uWT && g.ldwt % kLdAlign)))
        return hipErrorInvalidValue;
    } else {
      if ((epi != EPI_DGRAD && !g.bias) || (!g.C && !g.CT && !g.C2)) return hipErrorInvalidValue;
      if ((g.C && (g.ldc % kLdAlign || off(g.C))) || (g.CT && (g.ldct % kLdAlign || off(g.CT)))) return hipErrorInvalidValue;
      if (epi == EPI_DGRAD && g.maskT && (g.ldmask % kLdAlign || off(g.maskT))) return hipErrorInvalidValue;
    }
    if (epi == EPI_FWD_OUT) {
      const OutJob& o = group.out;
      if (p != 0 || !g.C || !o.dZ || !o.dZT || off(o.dZ) || off(o.dZT) || o.lddz % kLdAlign || o.lddzt % kLdAlign) return hipErrorInvalidValue;
      if (o.table ? (!o.y || !o.partials || !o.bad_ids || o.classes <= 0) : !o.ext) return hipErrorInvalidValue;
    }
    a.tile[p] = small_tile(dtype, g.M, g.N);
    a.tiles[p] = small_tile_count(dtype, g.M, g.N);
    a.first[p] = round_up(next, kXcds);
    next = a.first[p] + a.tiles[p];
    if (a.tile[p] == 64) lds = kLds64;
  }
  for (int p = 0; p < 2; ++p) {
    a.bias_first[p] = next;
    if (p < group.n_bias) next += (group.bias[p].N + 3) / 4;
  }
  a.sum_first = next;
  if (group.has_sum) next += 1;
  a.copy_first = next;
  if (group.has_copy) {
    const CopyJob& c = group.copy;
    if (off(c.in) || off(c.out) || off(c.outT) || c.ldin % ch || (c.out && c.ldo % ch) || (c.outT && (c.ldt % ch || c.rows_t % ch)))
      return hipErrorInvalidValue;
    next += ((c.C + 63) / 64) * ((c.R + 63) / 64);
  }
  hipError_t e = dtype == 1 ? configure<bf16>() : configure<float>();
  if (e != hipSuccess) return e;
  const bool alone = group.n == 1 && group.n_bias == 0 && !group.has_sum && !group.has_copy;
  if (alone && group.epi[0] == EPI_FWD)
    return dtype == 1 ? launch_product<bf16, EPI_FWD>(a.s.g[0], a.tile[0], a.tiles[0], s) : launch_product<float, EPI_FWD>(a.s.g[0], a.tile[0], a.tiles[0], s);
  if (alone && group.epi[0] == EPI_DGRAD)
    return dtype == 1 ? launch_product<bf16, EPI_DGRAD>(a.s.g[0], a.tile[0], a.tiles[0], s) : launch_product<float, EPI_DGRAD>(a.s.g[0], a.tile[0], a.tiles[0], s);
  if (dtype == 1) small_group_kernel<bf16><<<next, 256, lds, s>>>(a);
  else small_group_kernel<float><<<next, 256, lds, s>>>(a);
  return hipGetLastError();
}

}  // namespace slp
