// Device helpers of the memory-bound kernels (elementwise.hip) that the kernel for small layers (gemm_small.hip) also runs,
// in the same launch as its products.
#pragma once

#include "slp_kernels.h"

namespace slp {
namespace {

typedef __bf16 bf16;

template <typename T> __device__ __forceinline__ float to_f32(T v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v) { return (T)v; }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

// ---------------------------------------------------------------------------------
// 64x64 element tiles moved as 16-byte vectors
// ---------------------------------------------------------------------------------
// A tile row is CPR = 64/V chunks of V elements (V = 8 bf16 / 4 float).  Row-major traffic: lane -> (row,
// chunk) with the chunk index fastest, so a wavefront touches whole 128-byte row segments.  Transposed
// traffic: lane -> (column, chunk of V consecutive rows) with the row chunk fastest, the V values gathered
// from LDS.  In LDS, chunk ch of row r sits at chunk position ch ^ ((r / V) mod CPR): the row-major writes
// stay permutations within a row, and the gather of one wavefront instruction -- V-row groups 0..CPR-1 of a
// few adjacent columns -- lands in distinct banks.
template <typename T> struct Vec16;
template <> struct Vec16<bf16> { typedef __attribute__((ext_vector_type(8))) __bf16 type; static constexpr int n = 8; };
template <> struct Vec16<float> { typedef __attribute__((ext_vector_type(4))) float type; static constexpr int n = 4; };

template <typename T, int TILE = 64>
__device__ __forceinline__ int tile_slot(int row, int chunk) {     // position of a chunk in the LDS tile, in chunks
  constexpr int V = Vec16<T>::n, CPR = TILE / V;
  return row * CPR + (chunk ^ ((row / V) & (CPR - 1)));
}

// Writes the transposed tile: outT[c0 + c][r0 + r] for r below rows_t, from the LDS tile.
template <typename T, int TILE = 64>
__device__ __forceinline__ void store_tile_transposed(const typename Vec16<T>::type* tile, T* __restrict__ outT, int ldt,
                                                      int r0, int c0, int rows_t, int C) {
  typedef typename Vec16<T>::type vec_t;
  constexpr int V = Vec16<T>::n, CPR = TILE / V, ITEMS = TILE * CPR / 256;
  const T* flat = (const T*)tile;
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int idx = threadIdx.x + it * 256;
    const int cl = idx / CPR, rc = idx % CPR;
    const int c = c0 + cl, rs = r0 + rc * V;
    if (c < C && rs < rows_t) {
      vec_t o;
#pragma unroll
      for (int e = 0; e < V; ++e) o[e] = flat[tile_slot<T, TILE>(rc * V + e, cl / V) * V + (cl % V)];
      *(vec_t*)(outT + (size_t)c * ldt + rs) = o;
    }
  }
}

// Needs: in/out/mask 16-byte aligned with leading dimensions that are multiples of V (a chunk never straddles
// two rows; a chunk that straddles C reads pad elements of the same row, which callers keep allocated);
// rows_t (rows written to the transposed output) a multiple of V or beyond the data (pad rows are zeros).
// TILE x TILE elements per workgroup: 64 for small matrices (more workgroups), 128 for large bf16 ones (8 instead of 2
// vectors in flight per lane and 256-byte row segments on both sides: 8192 x 16384 in 0.20 -> see the launcher).
template <typename T, int TILE>
__device__ __forceinline__ void copy_transpose_block(int bx, int by, typename Vec16<T>::type* tile, const T* __restrict__ in, int ldin,
                                                     int R, int C, T* __restrict__ out, int ldo, T* __restrict__ outT, int ldt,
                                                     int rows_t, const T* __restrict__ mask, int ldmask) {
  typedef typename Vec16<T>::type vec_t;
  constexpr int V = Vec16<T>::n, CPR = TILE / V, ITEMS = TILE * CPR / 256;
  const int r0 = by * TILE, c0 = bx * TILE;
  vec_t v[ITEMS];
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {       // every load of the lane is issued before the first store
    const int idx = threadIdx.x + it * 256;
    const int row = idx / CPR, ch = idx % CPR;
    const int r = r0 + row, c = c0 + ch * V;
#pragma unroll
    for (int e = 0; e < V; ++e) v[it][e] = from_f32<T>(0.0f);
    if (r < R && c < C) {
      v[it] = *(const vec_t*)(in + (size_t)r * ldin + c);
      if (mask) {     // optional ReLU mask: the element passes only where mask[r][c] > 0
        const vec_t mk = *(const vec_t*)(mask + (size_t)r * ldmask + c);
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (!(to_f32<T>(mk[e]) > 0.0f)) v[it][e] = from_f32<T>(0.0f);
      }
#pragma unroll
      for (int e = 0; e < V; ++e)
        if (c + e >= C) v[it][e] = from_f32<T>(0.0f);     // pads stay zero
    }
  }
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int idx = threadIdx.x + it * 256;
    const int row = idx / CPR, ch = idx % CPR;
    const int r = r0 + row, c = c0 + ch * V;
    if (out && r < R && c < C) *(vec_t*)(out + (size_t)r * ldo + c) = v[it];
    tile[tile_slot<T, TILE>(row, ch)] = v[it];
  }
  if (!outT) return;
  __syncthreads();
  store_tile_transposed<T, TILE>(tile, outT, ldt, r0, c0, rows_t, C);
}

// ---------------------------------------------------------------------------------
// bias gradient: row sums of dZ^T, one wavefront per output feature
// ---------------------------------------------------------------------------------
// then the bias's own momentum update: v = mu v + db; b -= lr v (the gradient is kept for inspection)
template <typename T>
__device__ __forceinline__ void bias_grad_update_block(int block, const T* __restrict__ dZT, int ldt, int N, int B,
                                                       float* __restrict__ db, float* __restrict__ b,
                                                       float* __restrict__ vb, float lr, float mu) {
  constexpr int V = 16 / sizeof(T);
  typedef T vec_t __attribute__((ext_vector_type(V)));
  const int lane = threadIdx.x & 63;
  const int n = block * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  const T* row = dZT + (size_t)n * ldt;
  const int Bv = (B + V - 1) / V;      // pads up to the chunk boundary are zero
  // four independent 16-byte loads per lane and trip, so that the row streams instead of crawling load by load;
  // the partial sums are added in a fixed order
  float a4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int c0 = lane; c0 < Bv; c0 += 256) {
    vec_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + 64 * u;
      if (c < Bv) v[u] = *(const vec_t*)(row + (size_t)c * V);
      else
#pragma unroll
        for (int e = 0; e < V; ++e) v[u][e] = from_f32<T>(0.0f);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < V; ++e) a4[u] += to_f32((T)v[u][e]);
  }
  float acc = wave_sum((a4[0] + a4[1]) + (a4[2] + a4[3]));
  if (lane == 0) {
    db[n] = acc;
    float v = acc;
    if (mu != 0.0f) {
      v = mu * vb[n] + v;
      vb[n] = v;
    }
    b[n] -= lr * v;
  }
}

// out = scale * sum(partials), summed in double in a fixed order by one block of 256 threads
__device__ __forceinline__ void reduce_loss_block(double* red, const float* __restrict__ partials, int n, double scale, float* out0,
                                                  float* out1) {
  double acc = 0.0;
#pragma unroll 8      // the loads of 8 trips go out together (8192 x 16384: 47 us one by one); the order of the sum is the same
  for (int i = threadIdx.x; i < n; i += 256) acc += (double)partials[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const float v = (float)(red[0] * scale);
    out0[0] = v;
    if (out1) out1[0] = v;
  }
}

// Cross-entropy of four rows m0 .. m0 + 3 by one wavefront, whose lane holds logits zv[i][r] of columns lane + 64 i (past C: anything): losses,
// gradient row-major and, one vector of the four rows per column, transposed (dZT may be null).  at(r, id): logit id of row r.
template <typename T, int NC, typename At>
__device__ __forceinline__ void xent_rows(const float (&zv)[NC][4], int (&cls)[4], At at, int m0, int B, int C, int relu_last, float inv_b,
                                          T* __restrict__ dZ, int ld, T* __restrict__ dZT, int ldt, float* __restrict__ row_loss,
                                          unsigned* __restrict__ bad_ids) {
  typedef T vec4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & 63;
  float mx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY}, sum[4] = {0.0f, 0.0f, 0.0f, 0.0f}, lse[4];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    if (lane + 64 * i < C)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx[r] = fmaxf(mx[r], zv[i][r]);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) mx[r] = wave_max(mx[r]);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    if (lane + 64 * i < C)
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[r] += expf(zv[i][r] - mx[r]);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    sum[r] = wave_sum(sum[r]);
    lse[r] = mx[r] + logf(sum[r]);
    const int id = min(max(cls[r], 0), C - 1);
    if (lane == 0 && m0 + r < B) {
      if (id != cls[r]) atomicAdd(bad_ids, 1u);
      row_loss[m0 + r] = lse[r] - at(r, id);
    }
    cls[r] = id;
  }
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = lane + 64 * i;
    if (c < C) {
      vec4 g;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float zc = zv[i][r];
        const float p = expf(zc - lse[r]);
        const float d = (p - (c == cls[r] ? 1.0f : 0.0f)) * inv_b;
        g[r] = from_f32<T>((m0 + r >= B || (relu_last && !(zc > 0.0f))) ? 0.0f : d);
        if (m0 + r < B) dZ[(size_t)(m0 + r) * ld + c] = g[r];
      }
      if (dZT) *(vec4*)(dZT + (size_t)c * ldt + m0) = g;
    }
  }
}

}  // namespace
}  // namespace slp
