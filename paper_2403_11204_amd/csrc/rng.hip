// Seeded synthetic intermediate labels (paper Sec. 2, Eq. 1), the noisy label
// inputs of interior segments in the simultaneous variant (Sec. 2) and initial
// weights, all from one counter-based generator: Philox4x32-10 (Salmon et al.,
// SC'11) with key = seed and one counter per element, so that every value is a
// pure function of its coordinates and any launch shape gives the same bits.
//
// Counter convention:   labels   (i, class, 0, 0)
//                       weights  (in, out, 1, layer), bias at in = fan_in
//                       noise    (i, n_lo, 2, n_hi),  n = global sample index
//
// The float transforms are written as individually rounded IEEE float32
// operations (this file is compiled with floating-point contraction off, and the
// explicitly rounded intrinsics are used where a product feeds a sum) so that a
// CPU evaluating the same sequence gets the same bits.
#include "slp_kernels.h"

namespace slp {
namespace {

// a ^ b ^ c in one instruction (truth table 0x96)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96);
}

struct Words { uint32_t r0, r1; };      // the two words of a counter's four that the transforms use

constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u, kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;     // multipliers, Weyl sequence of the key

// One 32x32 -> 64 bit product per multiplier (v_mad_u64_u32) instead of a high-half and a low-half product each.  Rounds FIRST .. 9.
template <int FIRST = 0>
__device__ __forceinline__ Words philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                               uint32_t k1) {
#pragma unroll
  for (int round = FIRST; round < 10; ++round) {
    const uint64_t p0 = (uint64_t)kM0 * c0, p1 = (uint64_t)kM1 * c2;
    const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0 + round * kW0), n2 = xor3((uint32_t)(p0 >> 32), c3, k1 + round * kW1);
    c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
  }
  return Words{c0, c1};
}

// The counter is (column, row, stream, high word), and three rounds pass before column and row have met in every word.  Of their six products
// three depend on the column alone and are computed once for all rows that a lane takes of it, two on what a wavefront shares (stream, row) and
// are on the scalar unit, and one is left for every element.
struct ColumnPart { uint32_t x2, x0, y2, c3; };
__device__ __forceinline__ ColumnPart column_part(uint32_t column, uint32_t stream, uint32_t high, uint32_t k0, uint32_t k1) {
  const uint64_t a = (uint64_t)kM0 * column;                                                    // round 1, word 0
  const uint64_t b = (uint64_t)kM1 * xor3((uint32_t)(a >> 32), high, k1);                       // round 2, word 2
  const uint64_t c = (uint64_t)kM0 * xor3((uint32_t)(b >> 32), kM1 * stream, k0 + kW0);         // round 3, word 0
  return ColumnPart{(uint32_t)a, (uint32_t)b ^ (k0 + 2 * kW0), (uint32_t)(c >> 32) ^ (k1 + 2 * kW1), (uint32_t)c};
}
struct RowPart { uint32_t x2, y2; };
__device__ __forceinline__ RowPart row_part(uint32_t row, uint32_t stream, uint32_t k0, uint32_t k1) {
  const uint64_t a = (uint64_t)kM0 * ((uint32_t)(((uint64_t)kM1 * stream) >> 32) ^ row ^ k0);   // round 2, word 0
  return RowPart{(uint32_t)(a >> 32) ^ (k1 + kW1), (uint32_t)a};
}
__device__ __forceinline__ Words philox_of(const ColumnPart& c, const RowPart& r, uint32_t k0, uint32_t k1) {
  const uint64_t p = (uint64_t)kM1 * (c.x2 ^ r.x2);                                             // round 3, word 2
  return philox4x32_10<3>((uint32_t)(p >> 32) ^ c.x0, (uint32_t)p, c.y2 ^ r.y2, c.c3, k0, k1);
}

// IEEE square root: the plain builtin is lowered to the correctly rounded sequence
// (this file is built with -fhip-fp32-correctly-rounded-divide-sqrt); the
// "__fsqrt_rn" spelling maps to the 1-ulp native instruction and must not be used.
__device__ __forceinline__ float correctly_rounded_sqrt(float x) { return __builtin_sqrtf(x); }

// The same without the general sequence's scaling and special cases, for zeros and values in [2^-24, 64] (all that the
// normal transform asks for): the 1-ulp instruction, then one neighbour up or down where the sign of the residual, one
// fused operation each, says that it is the nearer one (Tuckerman's rounding test).  Correctly rounded from any estimate within 1
// ulp, for every significand of either parity of the exponent (tests/test_generator_rounding.py).
__device__ __forceinline__ float sqrt_unscaled(float x) {
  const float r = __builtin_amdgcn_sqrtf(x);
  const float lo = __uint_as_float(__float_as_uint(r) - 1u), hi = __uint_as_float(__float_as_uint(r) + 1u);
  float out = __fmaf_rn(-lo, r, x) <= 0.0f ? lo : r;
  out = __fmaf_rn(-hi, r, x) > 0.0f ? hi : out;
  return out;
}

// Correctly rounded a / d for d in [1.7, 2.5] and |a| < 1 (no scaling needed): a reciprocal refined once by Newton's step,
// the quotient corrected by its fused residual (Markstein 1990).  Correctly rounded from any reciprocal within 1 ulp, for every
// pair that ln_unit asks for (the same test).
__device__ __forceinline__ float divide_unscaled(float a, float d) {
  float y = __builtin_amdgcn_rcpf(d);
  y = __fmaf_rn(__fmaf_rn(-d, y, 1.0f), y, y);
  const float q = __fmul_rn(a, y);
  return __fmaf_rn(__fmaf_rn(-d, q, a), y, q);
}

__device__ __forceinline__ float unit_uniform(uint32_t r) {   // (r >> 8) * 2^-24, exact
  return __fmul_rn((float)(r >> 8), 0x1p-24f);
}

// ln(j * 2^-24), j in [1, 2^24]: mantissa/exponent split on the bit pattern of j (significand m in (sqrt(1/2), sqrt(2)]),
// atanh series in s = (m-1)/(m+1) to s^9, Horner with separately rounded
// multiplies and adds; exponent contribution split into a high and a low part.
__device__ __forceinline__ float ln_unit(uint32_t j) {
  const uint32_t bits = __float_as_uint((float)j) + (0x3F800000u - 0x3F3504F4u);   // significands above sqrt(2) carry
  const float ef = (float)((int)(bits >> 23) - (127 + 24));
  const float m = __uint_as_float((bits & 0x007FFFFFu) + 0x3F3504F4u);
  const float s = divide_unscaled(__fsub_rn(m, 1.0f), __fadd_rn(m, 1.0f));
  const float s2 = __fmul_rn(s, s);
  float p = __fadd_rn(__fmul_rn(s2, __uint_as_float(0x3E638E39u)), __uint_as_float(0x3E924925u));   // 2/9, 2/7
  p = __fadd_rn(__fmul_rn(p, s2), __uint_as_float(0x3ECCCCCDu));                                     // 2/5
  p = __fadd_rn(__fmul_rn(p, s2), __uint_as_float(0x3F2AAAABu));                                     // 2/3
  const float lnm = __fadd_rn(__fmul_rn(s, 2.0f), __fmul_rn(__fmul_rn(s, s2), p));
  return __fadd_rn(__fmul_rn(ef, __uint_as_float(0x3F317200u)),
                   __fadd_rn(__fmul_rn(ef, __uint_as_float(0x35BFBE8Eu)), lnm));
}

// cos(2 pi k / 2^24) for k = r >> 8: exact quadrant and reflection in integers,
// then Taylor polynomials of sin and cos on [0, pi/4].
__device__ __forceinline__ float cos_turn(uint32_t r) {
  const uint32_t fi = (r >> 8) & 0x3FFFFFu;
  const bool swap = fi > (1u << 21);
  const uint32_t ti = swap ? (1u << 22) - fi : fi;
  const float x = __fmul_rn((float)ti, 0x1.921FB6p+0f * 0x1p-22f);     // pi/2 * 2^-22: the scaling is exact
  const float x2 = __fmul_rn(x, x);
  float sp = __fadd_rn(__fmul_rn(x2, __uint_as_float(0x3638EF1Du)), __uint_as_float(0xB9500D01u));
  sp = __fadd_rn(__fmul_rn(sp, x2), __uint_as_float(0x3C088889u));
  sp = __fadd_rn(__fmul_rn(sp, x2), __uint_as_float(0xBE2AAAABu));
  const float sinx = __fadd_rn(x, __fmul_rn(__fmul_rn(x, x2), sp));
  float cp = __fadd_rn(__fmul_rn(x2, __uint_as_float(0xB493F27Eu)), __uint_as_float(0x37D00D01u));
  cp = __fadd_rn(__fmul_rn(cp, x2), __uint_as_float(0xBAB60B61u));
  cp = __fadd_rn(__fmul_rn(cp, x2), __uint_as_float(0x3D2AAAABu));
  cp = __fadd_rn(__fmul_rn(cp, x2), -0.5f);
  const float cosx = __fadd_rn(1.0f, __fmul_rn(x2, cp));
  // quadrants 0..3 (the top two bits): cos, -sin, -cos, sin of the quadrant's angle, which reflection exchanges
  const float v = (swap != (bool)((r >> 30) & 1u)) ? sinx : cosx;
  return __uint_as_float(__float_as_uint(v) ^ ((r ^ (r << 1)) & 0x80000000u));
}

__device__ __forceinline__ float standard_normal(uint32_t r0, uint32_t r1) {
  const float radius = sqrt_unscaled(__fmul_rn(-2.0f, ln_unit((r0 >> 8) + 1u)));
  return __fmul_rn(radius, cos_turn(r1));
}

template <int DIST>
__device__ __forceinline__ float draw(float kappa, const Words& w) {
  if (DIST == 0) return __fmul_rn(kappa, unit_uniform(w.r0));
  if (DIST == 1) return __fsub_rn(__fmul_rn(2.0f, unit_uniform(w.r0)), 1.0f);
  if (DIST == 2) return standard_normal(w.r0, w.r1);
  return (w.r0 >> 31) ? 1.0f : -1.0f;
}

__device__ __forceinline__ void store_value(float* out, size_t idx, float v) { out[idx] = v; }
// round to nearest even in one instruction; NaN keeps its upper bits and becomes quiet
__device__ __forceinline__ void store_value(__bf16* out, size_t idx, float v) { out[idx] = (__bf16)v; }

// Every kernel here is bound by its integer and float instructions (10 rounds of two 64-bit products, then the transform),
// not by the bytes it writes.  A wavefront therefore takes a run of kRun columns of ONE row, column by column across its
// lanes: the row's index is uniform over the wavefront, so the division that finds it and every part of the counter
// arithmetic that depends on the row and the key only is done once per run on the scalar unit, and the stores are
// coalesced whatever the alignment of a row.  fn(row, column) is called for every element, whole runs without a test per column.
// 8192 x 16384 bf16 inputs and their 1000 x 16384 table, both calls: one element per lane with a 64-bit division each, the
// general division and square root and separate halves of the products 564 us -> 323 us (with several rows per wavefront, below, 293); what is
// left is issued at the rate of the vector units.  Unrolled by 4: by 2 +5 %, by 8 the same.
// Rows of up to kFlat columns leave too many lanes without one and pay for the row too often: there a wavefront takes kFlat elements
// as they lie, over the rows' ends; one division on the scalar unit for the first, by 2^32 / cols for the others.  200000 rows of
// float32 inputs, microseconds, one element per lane as before / a run per row (up to 32 columns several rows per wavefront) / this:
// 17 columns 19.5 / 23.9 / 14.9, 33 33.3 / 50.2 / 25.0, 47 45.6 / 51.5 / 32.9, 60 57 / 51 / 40, 65 61 / 72 / 43, 72 67 / 73 / 47;
// 300 232 / 157 / 178.
constexpr int kRun = 512, kFlat = 256;
template <typename F>
__device__ __forceinline__ void for_each_element(uint32_t rows, uint32_t cols, uint32_t reciprocal, F fn) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t waves = (uint64_t)gridDim.x * 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (reciprocal) {
    const uint64_t total = (uint64_t)rows * cols;
    for (uint64_t u = (uint64_t)blockIdx.x * 4 + wave; u * kFlat < total; u += waves) {
      const uint64_t first = u * kFlat, left = total - first;
      const uint32_t r0 = total >> 32 ? (uint32_t)(first / cols) : (uint32_t)first / cols, c0 = (uint32_t)(first - (uint64_t)r0 * cols);
#pragma unroll
      for (uint32_t j = 0; j < kFlat; j += 64)
        if (j + lane < left) {
          const uint32_t e = c0 + j + lane;                     // below cols + kFlat: the quotient is at most one too small
          uint32_t q = __umulhi(e, reciprocal), c = e - q * cols;
          if (c >= cols) { ++q; c -= cols; }
          fn(r0 + q, c);
        }
    }
    return;
  }
  const uint32_t runs = (cols + kRun - 1) / kRun;
  const uint64_t units = (uint64_t)rows * runs;
  for (uint64_t u = (uint64_t)blockIdx.x * 4 + wave; u < units; u += waves) {
    const uint32_t r = (uint32_t)(u / runs), c0 = (uint32_t)(u % runs) * kRun;
    if (cols - c0 >= kRun) {
#pragma unroll 4
      for (int j = 0; j < kRun / 64; ++j) fn(r, c0 + 64 * j + lane);
    } else {
      for (uint32_t c = c0 + lane; c < cols; c += 64) fn(r, c);
    }
  }
}

// Large matrices (see rows_per_wave): a wavefront takes kDeepRun columns of `deep` rows, and the columns' share of the counter arithmetic stays in
// registers from row to row: for inputs 14 products and 13 three-way xors an element instead of 17 and 18.
// fn(row, column, words of the counter); low(row), high(row) give the row's words of the counter.
constexpr int kDeepRun = 256;
template <typename L, typename H, typename F>
__device__ __forceinline__ void for_each_of_rows(uint32_t rows, uint32_t cols, uint32_t deep, uint32_t stream, uint32_t k0, uint32_t k1, L low, H high, F fn) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t waves = (uint64_t)gridDim.x * 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t runs = (cols + kDeepRun - 1) / kDeepRun;
  const uint64_t units = (uint64_t)((rows + deep - 1) / deep) * runs;
  for (uint64_t u = (uint64_t)blockIdx.x * 4 + wave; u < units; u += waves) {
    const uint32_t r0 = (uint32_t)(u / runs) * deep, c0 = (uint32_t)(u % runs) * kDeepRun;
    const uint32_t r1 = rows - r0 < deep ? rows : r0 + deep;
    ColumnPart cp[kDeepRun / 64];
    uint32_t h = high(r0);
    auto columns = [&]() {
#pragma unroll
      for (int j = 0; j < kDeepRun / 64; ++j) cp[j] = column_part(c0 + 64 * j + lane, stream, h, k0, k1);
    };
    columns();
    const bool whole = cols - c0 >= kDeepRun;
    for (uint32_t r = r0; r < r1; ++r) {
      if (high(r) != h) {          // the row's index went past 2^32
        h = high(r);
        columns();
      }
      const RowPart rp = row_part(low(r), stream, k0, k1);
      if (whole) {
#pragma unroll
        for (int j = 0; j < kDeepRun / 64; ++j) fn(r, c0 + 64 * j + lane, philox_of(cp[j], rp, k0, k1));
      } else {
#pragma unroll
        for (int j = 0; j < kDeepRun / 64; ++j)
          if (c0 + 64 * j + lane < cols) fn(r, c0 + 64 * j + lane, philox_of(cp[j], rp, k0, k1));
      }
    }
  }
}

template <typename T, int DIST>
__global__ __launch_bounds__(256) void labels_kernel(uint32_t k0, uint32_t k1, int classes, int dim, float kappa, T* __restrict__ out,
                                                     uint32_t reciprocal) {
  for_each_element(classes, dim, reciprocal, [&](uint32_t j, uint32_t i) {
    store_value(out, (size_t)j * dim + i, draw<DIST>(kappa, philox4x32_10(i, j, 0u, 0u, k0, k1)));
  });
}
template <typename T, int DIST>
__global__ __launch_bounds__(256) void labels_rows_kernel(uint32_t k0, uint32_t k1, int classes, int dim, float kappa, T* __restrict__ out,
                                                          uint32_t deep) {
  for_each_of_rows(classes, dim, deep, 0u, k0, k1, [](uint32_t j) { return j; }, [](uint32_t) { return 0u; },
                   [&](uint32_t j, uint32_t i, const Words& w) { store_value(out, (size_t)j * dim + i, draw<DIST>(kappa, w)); });
}

template <typename T>
__device__ __forceinline__ void store_input(const float* __restrict__ table, int classes, const int32_t* __restrict__ y, uint32_t row, int dim, uint32_t i,
                                            float sigma, const Words& w, T* __restrict__ out) {
  const float z = standard_normal(w.r0, w.r1);
  const int cls = min(max(y[row], 0), classes - 1);
  const float v = __fadd_rn(table[(size_t)cls * dim + i], __fmul_rn(sigma, z));
  store_value(out, (size_t)row * dim + i, v);
}
template <typename T>
__global__ __launch_bounds__(256) void inputs_kernel(uint32_t k0, uint32_t k1, const float* __restrict__ table, int classes,
                                                     const int32_t* __restrict__ y, uint64_t first, int batch, int dim, float sigma,
                                                     T* __restrict__ out, uint32_t reciprocal) {
  for_each_element(batch, dim, reciprocal, [&](uint32_t row, uint32_t i) {
    const uint64_t n = first + row;
    store_input(table, classes, y, row, dim, i, sigma, philox4x32_10(i, (uint32_t)n, 2u, (uint32_t)(n >> 32), k0, k1), out);
  });
}
template <typename T>
__global__ __launch_bounds__(256) void inputs_rows_kernel(uint32_t k0, uint32_t k1, const float* __restrict__ table, int classes,
                                                          const int32_t* __restrict__ y, uint64_t first, int batch, int dim, float sigma,
                                                          T* __restrict__ out, uint32_t deep) {
  for_each_of_rows(batch, dim, deep, 2u, k0, k1, [&](uint32_t row) { return (uint32_t)(first + row); }, [&](uint32_t row) { return (uint32_t)((first + row) >> 32); },
                   [&](uint32_t row, uint32_t i, const Words& w) { store_input(table, classes, y, row, dim, i, sigma, w, out); });
}

__device__ __forceinline__ void store_weight(float* __restrict__ W, int K, int ldk, float* __restrict__ b, uint32_t o, uint32_t k, float bound, const Words& w) {
  const float v = __fmul_rn(__fsub_rn(__fmul_rn(2.0f, unit_uniform(w.r0)), 1.0f), bound);
  if ((int)k < K) W[(size_t)o * ldk + k] = v;
  else b[o] = v;
}
__global__ __launch_bounds__(256) void init_kernel(uint32_t k0, uint32_t k1, uint32_t layer, float* __restrict__ W, int N, int K,
                                                   int ldk, float* __restrict__ b, uint32_t reciprocal) {
  const float bound = __fdiv_rn(1.0f, correctly_rounded_sqrt((float)K));
  for_each_element(N, (uint32_t)K + 1, reciprocal,
                   [&](uint32_t o, uint32_t k) { store_weight(W, K, ldk, b, o, k, bound, philox4x32_10(k, o, 1u, layer, k0, k1)); });
}
__global__ __launch_bounds__(256) void init_rows_kernel(uint32_t k0, uint32_t k1, uint32_t layer, float* __restrict__ W, int N, int K,
                                                        int ldk, float* __restrict__ b, uint32_t deep) {
  const float bound = __fdiv_rn(1.0f, correctly_rounded_sqrt((float)K));
  for_each_of_rows(N, (uint32_t)K + 1, deep, 1u, k0, k1, [](uint32_t o) { return o; }, [&](uint32_t) { return layer; },
                   [&](uint32_t o, uint32_t k, const Words& w) { store_weight(W, K, ldk, b, o, k, bound, w); });
}

// 2^32 / cols, rounded down, for rows of up to kFlat columns; 0 for others
inline uint32_t reciprocal_for(size_t cols) { return cols <= (size_t)kFlat ? (uint32_t)(0xFFFFFFFFu / cols) : 0u; }
inline int blocks_of(size_t units) {            // of 4 wavefronts; above 2^18 of them the kernels loop
  const size_t blocks = (units + 3) / 4;
  return (int)(blocks < 1 ? 1 : (blocks > (1u << 18) ? (1u << 18) : blocks));
}
inline int grid_for(size_t rows, size_t cols) {
  return blocks_of(cols <= (size_t)kFlat ? (rows * cols + kFlat - 1) / kFlat : rows * ((cols + kRun - 1) / kRun));
}
inline int grid_of_rows(size_t rows, size_t cols, uint32_t deep) { return blocks_of((rows + deep - 1) / deep * ((cols + kDeepRun - 1) / kDeepRun)); }

// Rows per wavefront of for_each_of_rows; 0: for_each_element.  So many that every SIMD still has eight wavefronts or more, and only where the last
// run of a row has most of its columns: a lane past them idles for all rows.  Microseconds, one row / 2 / 4 / 8 (/ 16), bf16 normal labels (bf16
// inputs): 1000 x 2048 (8000 runs of kDeepRun columns) 7.0 / 7.3 / 7.5 / 9.3, 4096 x 1000 (16384) 12.7 / 12.5 / 12.4 / 13.2 (13.3 / 12.8 / 12.9 / 14.5),
// 8192 x 768 (24576) 18.1 / 17.4 / 16.8 / 17.6, 20000 x 768 (60000) 39.6 / 38.1 / 36.4 / 38.7, float32 uniform ones 1000 x 16384 (64000) 22.2 / 21.6 /
// 20.0 / 19.3, 2000 x 16384 (128000) 74.8 / 75.8 / 72.7 / 71.6 (77.1 / 74.5 / 73.0 / 72.0), 8192 x 16384 (524288)
// 292 / 298 / 287 / 285 / 283 (310 / 309 / 297 / 294 / 288); a last run of 1 column of 256 in 5 runs, 8192 x 1025, 28.2 / 26.2 / 25.7 / 26.0, of 88 in 3, 8192 x 600,
// 16.2 / 16.9 / 16.6 / 17.4, of 1 in 3, 8192 x 513, 14.7 / 17.0 / 16.6 / 17.5.
inline uint32_t rows_per_wave(size_t rows, size_t cols) {
  const size_t runs = (cols + kDeepRun - 1) / kDeepRun, total = rows * runs;
  if (cols <= (size_t)kFlat || 4 * runs * kDeepRun > 5 * cols || total < 16384) return 0;
  return total < 24576 ? 2 : (total < 62000 ? 4 : (total < 262144 ? 8 : 16));
}

template <typename T, int DIST>
void launch_labels_of(uint32_t k0, uint32_t k1, int classes, int dim, float kappa, T* out, hipStream_t s) {
  if (const uint32_t deep = rows_per_wave(classes, dim))
    labels_rows_kernel<T, DIST><<<grid_of_rows(classes, dim, deep), 256, 0, s>>>(k0, k1, classes, dim, kappa, out, deep);
  else
    labels_kernel<T, DIST><<<grid_for(classes, dim), 256, 0, s>>>(k0, k1, classes, dim, kappa, out, reciprocal_for(dim));
}
template <typename T>
void launch_labels(uint64_t seed, int classes, int dim, int dist, float kappa, T* out, hipStream_t s) {
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  switch (dist) {
    case 0: launch_labels_of<T, 0>(k0, k1, classes, dim, kappa, out, s); break;
    case 1: launch_labels_of<T, 1>(k0, k1, classes, dim, kappa, out, s); break;
    case 2: launch_labels_of<T, 2>(k0, k1, classes, dim, kappa, out, s); break;
    default: launch_labels_of<T, 3>(k0, k1, classes, dim, kappa, out, s); break;
  }
}
template <typename T>
void launch_inputs(uint64_t seed, const float* table, int classes, const int32_t* y, int64_t first_sample, int batch, int dim, float sigma, T* out,
                   hipStream_t s) {
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  if (const uint32_t deep = rows_per_wave(batch, dim))
    inputs_rows_kernel<<<grid_of_rows(batch, dim, deep), 256, 0, s>>>(k0, k1, table, classes, y, (uint64_t)first_sample, batch, dim, sigma, out, deep);
  else
    inputs_kernel<<<grid_for(batch, dim), 256, 0, s>>>(k0, k1, table, classes, y, (uint64_t)first_sample, batch, dim, sigma, out, reciprocal_for(dim));
}

}  // namespace

hipError_t launch_make_labels(uint64_t seed, int classes, int dim, int dist, float kappa, void* out, int dt,
                              hipStream_t s) {
  if (dt == 1) launch_labels(seed, classes, dim, dist, kappa, (__bf16*)out, s);
  else launch_labels(seed, classes, dim, dist, kappa, (float*)out, s);
  return hipGetLastError();
}

hipError_t launch_make_inputs(uint64_t seed, const float* table, int classes, const int32_t* y, int64_t first_sample,
                              int batch, int dim, float sigma, void* out, int dt, hipStream_t s) {
  if (dt == 1) launch_inputs(seed, table, classes, y, first_sample, batch, dim, sigma, (__bf16*)out, s);
  else launch_inputs(seed, table, classes, y, first_sample, batch, dim, sigma, (float*)out, s);
  return hipGetLastError();
}

hipError_t launch_init_weights(uint64_t seed, int layer, float* W32, int N, int K, int ldk, float* b, hipStream_t s) {
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  const size_t cols = (size_t)K + 1;
  if (const uint32_t deep = rows_per_wave(N, cols))
    init_rows_kernel<<<grid_of_rows(N, cols, deep), 256, 0, s>>>(k0, k1, (uint32_t)layer, W32, N, K, ldk, b, deep);
  else
    init_kernel<<<grid_for(N, cols), 256, 0, s>>>(k0, k1, (uint32_t)layer, W32, N, K, ldk, b, reciprocal_for(cols));
  return hipGetLastError();
}

}  // namespace slp
