// Memory-bound kernels of the segment step: input ingest / transposes, the two
// loss kernels (paper Sec. 2: regression on the synthetic label of the sample's
// class for a non-final segment, classification for the final one), bias
// gradients and the SGD-with-momentum update (Sec. 3).  All are written for
// coalesced traffic (a wavefront touches consecutive addresses on both the read
// and the write side; transposes go through LDS) and reduce with wavefront
// shuffles in a fixed order, so results are bit-reproducible from run to run.
#include "elementwise_device.h"

namespace slp {
namespace {

// see copy_transpose_block
template <typename T, int TILE>
__global__ __launch_bounds__(256) void copy_transpose_vec_kernel(const T* __restrict__ in, int ldin, int R, int C,
                                                                 T* __restrict__ out, int ldo, T* __restrict__ outT,
                                                                 int ldt, int rows_t, const T* __restrict__ mask,
                                                                 int ldmask) {
  __shared__ typename Vec16<T>::type tile[TILE * TILE / Vec16<T>::n];
  copy_transpose_block<T, TILE>(blockIdx.x, blockIdx.y, tile, in, ldin, R, C, out, ldo, outT, ldt, rows_t, mask, ldmask);
}

// ---------------------------------------------------------------------------------
// copy + transpose through a 64x64 LDS tile, element by element (any alignment)
// ---------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void copy_transpose_kernel(const T* __restrict__ in, int ldin, int R, int C,
                                                             T* __restrict__ out, int ldo, T* __restrict__ outT,
                                                             int ldt, int pad_t, const T* __restrict__ mask,
                                                             int ldmask) {
  __shared__ T tile[64][65];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int rr = ty; rr < 64; rr += 4) {
    const int r = r0 + rr, c = c0 + tx;
    T v = from_f32<T>(0.0f);
    if (r < R && c < C) {
      v = in[(size_t)r * ldin + c];
      // optional ReLU mask: the element passes only where mask[r][c] > 0
      if (mask && !(to_f32(mask[(size_t)r * ldmask + c]) > 0.0f)) v = from_f32<T>(0.0f);
      if (out) out[(size_t)r * ldo + c] = v;
    }
    tile[rr][tx] = v;
  }
  if (!outT) return;
  __syncthreads();
  const int R8 = pad_t ? ((R + 7) & ~7) : R;
  for (int cc = ty; cc < 64; cc += 4) {
    const int c = c0 + cc, r = r0 + tx;
    if (c < C && r < R8) outT[(size_t)c * ldt + r] = tile[tx][cc];
  }
}

// ---------------------------------------------------------------------------------
// mean squared error against the synthetic label of each row's class
// ---------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void mse_loss_grad_kernel(const T* __restrict__ AL, int ld, const int32_t* __restrict__ y,
                                                            const float* __restrict__ table, int classes, int B, int D,
                                                            int relu_last,
                                                            float scale, T* __restrict__ dZ, T* __restrict__ dZT, int ldt,
                                                            float* __restrict__ partials, unsigned* __restrict__ bad_ids) {
  typedef typename Vec16<T>::type vec_t;
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  constexpr int V = Vec16<T>::n, CPR = 64 / V, ITEMS = 64 * CPR / 256;
  __shared__ vec_t tile[64 * CPR];
  __shared__ float red[4];
  const int b0 = blockIdx.y * 64, d0 = blockIdx.x * 64;
  const bool table_vec = (D & 3) == 0;        // label rows start 16-byte aligned
  float lsum = 0.0f;
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int idx = threadIdx.x + it * 256;
    const int row = idx / CPR, ch = idx % CPR;
    const int m = b0 + row, i = d0 + ch * V;
    vec_t gv;
#pragma unroll
    for (int e = 0; e < V; ++e) gv[e] = from_f32<T>(0.0f);
    if (m < B && i < D) {
      const vec_t av = *(const vec_t*)(AL + (size_t)m * ld + i);     // a chunk that straddles D reads pad zeros
      const int cls = min(max(y[m], 0), classes - 1);                 // ids are the caller's; never index outside the table
      if (cls != y[m] && blockIdx.x == 0 && ch == 0) atomicAdd(bad_ids, 1u);   // once per row; rare, and the count is an integer
      const float* trow = table + (size_t)cls * D + i;
      float tv[V];
      if (table_vec && i + V <= D) {
#pragma unroll
        for (int q = 0; q < V / 4; ++q) {
          const f32x4 t4 = *(const f32x4*)(trow + 4 * q);
#pragma unroll
          for (int e = 0; e < 4; ++e) tv[4 * q + e] = t4[e];
        }
      } else {
#pragma unroll
        for (int e = 0; e < V; ++e) tv[e] = i + e < D ? trow[e] : 0.0f;
      }
#pragma unroll
      for (int e = 0; e < V; ++e) {
        if (i + e < D) {
          const float a = to_f32<T>(av[e]);
          const float d = a - tv[e];
          lsum += d * d;
          gv[e] = from_f32<T>((relu_last && !(a > 0.0f)) ? 0.0f : scale * d);
        }
      }
      if (dZ) *(vec_t*)(dZ + (size_t)m * ld + i) = gv;
    }
    tile[tile_slot<T>(row, ch)] = gv;
  }
  lsum = wave_sum(lsum);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lsum;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.y * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
  store_tile_transposed<T>(tile, dZT, ldt, b0, d0, (B + 7) & ~7, D);
}

// ---------------------------------------------------------------------------------
// softmax cross-entropy
// ---------------------------------------------------------------------------------
// C <= 64 NC: four rows per wavefront, the logits read once and kept in registers.  A lane holds column c of four consecutive
// rows, so that it can store them into the transposed gradient as one vector of 8 or 16 bytes (a workgroup covers 16 rows, 32
// or 64 bytes of a line; the rest of it comes from other workgroups) and the four rows' reductions run side by side: what
// bounds this kernel at the sizes in use is their latency, not its bytes.  The order of each row's sum is that of one row per
// wavefront.  See launch_xent for where it is used.
template <typename T, int NC>
__global__ __launch_bounds__(256) void xent_loss_grad_kernel(const T* __restrict__ ZL, int ld, const int32_t* __restrict__ y,
                                                             int B, int C, int relu_last, float inv_b,
                                                             T* __restrict__ dZ, T* __restrict__ dZT, int ldt,
                                                             float* __restrict__ row_loss, unsigned* __restrict__ bad_ids) {
  typedef T vec4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & 63;
  const int m0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 4;
  if (m0 >= ((B + 7) & ~7)) return;
  const T* z[4];
  int cls[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = min(m0 + r, B - 1);          // rows past the batch read the last one and store zeros
    z[r] = ZL + (size_t)m * ld;
    cls[r] = y[m];
  }
  float zv[NC][4];
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) zv[i][r] = lane + 64 * i < C ? to_f32<T>(z[r][lane + 64 * i]) : -INFINITY;
  xent_rows<T, NC>(zv, cls, [&](int r, int id) { return to_f32<T>(z[r][id]); }, m0, B, C, relu_last, inv_b, dZ, ld, dZT, ldt, row_loss, bad_ids);
}

// Any number of classes: one row per wavefront, the logits read three times, and the transposed gradient by a launch of its own.
// Four rows per wavefront with three reads were a quarter of the wavefronts, each four times as long, and stored 16 rows' worth
// of a line at a time.  Microseconds, this kernel + transpose / four rows: float32 256 x 1000 13.6 + 4.2 / 30.3, 8192 x 1000
// 24.0 + 11.4 / 48.3, 8192 x 4096 106 + 43 / 249; bf16 8192 x 1000 22.0 + 6.8 / 44.5, 8192 x 4096 75.5 + 22.3 / 166.
template <typename T>
__global__ __launch_bounds__(256) void xent_loss_grad_wide_kernel(const T* __restrict__ ZL, int ld, const int32_t* __restrict__ y,
                                                                  int B, int C, int relu_last, float inv_b, T* __restrict__ dZ,
                                                                  float* __restrict__ row_loss, unsigned* __restrict__ bad_ids) {
  const int lane = threadIdx.x & 63;
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (m >= B) return;
  const T* z = ZL + (size_t)m * ld;
  float mx = -INFINITY;
  for (int c = lane; c < C; c += 64) mx = fmaxf(mx, to_f32<T>(z[c]));
  mx = wave_max(mx);
  float sum = 0.0f;
  for (int c = lane; c < C; c += 64) sum += expf(to_f32<T>(z[c]) - mx);
  sum = wave_sum(sum);
  const float lse = mx + logf(sum);
  const int cls = min(max(y[m], 0), C - 1);
  if (lane == 0) {
    if (cls != y[m]) atomicAdd(bad_ids, 1u);
    row_loss[m] = lse - to_f32<T>(z[cls]);
  }
  T* g = dZ + (size_t)m * ld;
  for (int c = lane; c < C; c += 64) {
    const float zc = to_f32<T>(z[c]);
    const float p = expf(zc - lse);
    const float d = (p - (c == cls ? 1.0f : 0.0f)) * inv_b;
    g[c] = from_f32<T>((relu_last && !(zc > 0.0f)) ? 0.0f : d);
  }
}

// out = scale * sum(partials), summed in double in a fixed order by one block.  (A separate launch on purpose:
// finishing the sum inside the loss kernels -- last block counted in by an atomic -- needs a device-scope fence per
// block, which on this chip writes back the whole L2 of the block's XCD: measured 25x slower than this launch.)
__global__ __launch_bounds__(256) void reduce_loss_kernel(const float* __restrict__ partials, int n, double scale,
                                                          float* out0, float* out1) {
  __shared__ double red[256];
  reduce_loss_block(red, partials, n, scale, out0, out1);
}

// ---------------------------------------------------------------------------------
// SGD with momentum on one weight matrix + derived copies
// ---------------------------------------------------------------------------------
// A block owns a 64 (out) x 64 (in) tile.  Every thread moves 16-byte vectors: four
// consecutive inputs of one output row for the float32 streams (gradient, momentum,
// master weight), and four consecutive outputs of one input row for the transposed copy,
// which goes through an LDS tile.  Pad columns (in >= K, up to the leading dimension) hold
// zeros in all three streams and stay zero under the update, so the row direction needs
// no tail handling.
template <typename T, bool REFRESH = false>      // REFRESH: no arithmetic, the copies are rebuilt from W32
__device__ __forceinline__ void sgd_update_block(int bx, int by, float* __restrict__ W32, float* __restrict__ vW,
                                                 const float* __restrict__ dW, int N, int K, int ldk,
                                                 bf16* __restrict__ W16, T* __restrict__ WT, int ldn, float lr,
                                                 float mu) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef T tx4 __attribute__((ext_vector_type(4)));
  typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
  __shared__ T tile[64][68];
  const int n0 = by * 64, k0 = bx * 64;
  const int q = threadIdx.x & 15, r = threadIdx.x >> 4;
  const int k = k0 + q * 4;
  // all loads of the thread's four rows are issued before the first store, so that 9 to 12
  // 16-byte requests per thread are in flight
  f32x4 w[4], gr[4], vo[4];
  const bool with_v = !REFRESH && mu != 0.0f;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int n = n0 + r + 16 * p;
    const bool in = n < N && k < K;
    const size_t idx = (size_t)n * ldk + k;
    w[p] = in ? __builtin_nontemporal_load((const f32x4*)(W32 + idx)) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    gr[p] = (in && !REFRESH) ? __builtin_nontemporal_load((const f32x4*)(dW + idx)) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    vo[p] = (in && with_v) ? __builtin_nontemporal_load((const f32x4*)(vW + idx)) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int rr = r + 16 * p, n = n0 + rr;
    if (n < N && k < K) {
      const size_t idx = (size_t)n * ldk + k;
      if (!REFRESH) {
        f32x4 v = gr[p];
        if (with_v) {
          v = mu * vo[p] + v;
          __builtin_nontemporal_store(v, (f32x4*)(vW + idx));
        }
        w[p] = w[p] - lr * v;
        __builtin_nontemporal_store(w[p], (f32x4*)(W32 + idx));
      }
      if (W16) {
        bf16x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = (bf16)w[p][e];
        *(bf16x4*)(W16 + idx) = h;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[rr][q * 4 + e] = from_f32<T>(w[p][e]);
  }
  if (!WT) return;      // (uniform over the launch)
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int kk = r + 16 * p, kg = k0 + kk, n = n0 + q * 4;
    if (kg < K && n < N) {
      tx4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = tile[q * 4 + e][kk];
      *(tx4*)(WT + (size_t)kg * ldn + n) = o;
    }
  }
}

// One launch updates a whole layer: blocks [0, kb*nb) each own a 64x64 tile of the weight matrix, the blocks after
// them 4 output features of the bias each (gradient = row sum of dZ^T, then the same momentum update).
struct LayerUpdate {
  float *W32, *vW; const float* dW; int N, K, ldk; void* W16; void* WT; int ldn;     // weights [N][ldk]
  const void* dZT; int ldt, B; float *db, *b, *vb;                                     // bias: dZT [N][ldt]; null = weights only
  float lr, mu;
};

// the copies alone, one block per 64x64 tile on a 2-D grid
template <typename T>
__global__ __launch_bounds__(256) void refresh_copies_kernel(float* __restrict__ W32, int N, int K, int ldk, bf16* __restrict__ W16,
                                                             T* __restrict__ WT, int ldn) {
  sgd_update_block<T, true>(blockIdx.x, blockIdx.y, W32, nullptr, nullptr, N, K, ldk, W16, WT, ldn, 0.0f, 0.0f);
}

// The update of the weight matrix alone on a fixed number of workgroups that walk the tiles with the grid's stride: for updates that run beside
// matrix products.  At full width the update saturates HBM and the product next to it, which waits on every load,
// all but stops (measured: a 1.3 ms update stretched the product beside it from 3.15 to 4.29 ms); one workgroup per
// compute unit takes longer over the same bytes and costs the product less.
// Held to 64 registers per lane (8 wavefronts per SIMD): the 256x256 product kernel's two wavefronts per SIMD, or the one of long
// contractions, take up to 448 of the 512 registers, and a wavefront that needs more than the 64 left cannot share the SIMD with them.  At 68 the
// update's workgroups could only start on a compute unit between two product workgroups and then kept the next one
// out for as long as they ran (comparison configuration: 38.9 -> 36.9 ms per step with the limit).
// pause: units of ~0.5 us that a workgroup sleeps after each 64x64 tile.  A compute unit's vector memory path delivers
// ~56 GB/s (measured with one copy workgroup per compute unit) and the product beside the update already takes ~48 of
// them, so the update's loads queue in front of the product's; spread over twice the time they fit into the headroom
// (comparison configuration 37.1 -> 36.7 ms per step, deep configuration run serially 13.2 -> 12.9 at 8-14 units; the
// update's tail must still find products to hide behind, which is why the caller sizes the pause by the batch).
// hurry: a flag that is raised on a stream that comes to wait for the update (hurry_kernel): from the next tile on nothing sleeps
// any more, what that stream ran beside the update is over.  (A second stream of the caller's may still have products in
// flight; they then share the chip with an update that does not pause.)  Only a
// launch that pauses reads the flag, once a tile.  A segment of 784-16384-16384-16384 stepped on its own waited 2.4 ms for the paced update of its second
// layer, 1.3 without the pauses.
template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void sgd_update_strided_kernel(float* __restrict__ W32, float* __restrict__ vW,
                                                                 const float* __restrict__ dW, int N, int K, int ldk,
                                                                 bf16* __restrict__ W16, T* __restrict__ WT, int ldn, float lr,
                                                                 float mu, int pause, const unsigned* hurry) {
  const int kb = (K + 63) / 64, tiles = kb * ((N + 63) / 64);
  for (int id = blockIdx.x; id < tiles; id += gridDim.x) {
    const unsigned h = pause > 0 ? __hip_atomic_load(hurry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    sgd_update_block<T>(id % kb, id / kb, W32, vW, dW, N, K, ldk, W16, WT, ldn, lr, mu);
    if (h) pause = 0;
    for (int i = 0; i < pause; ++i) __builtin_amdgcn_s_sleep(16);
    __syncthreads();   // the LDS tile is reused
  }
}

__global__ void hurry_kernel(unsigned* hurry, unsigned value) {
  __hip_atomic_store(hurry, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__global__ __launch_bounds__(256) void layer_update_kernel(const LayerUpdate u) {
  const int kb = (u.K + 63) / 64, nb = (u.N + 63) / 64;
  const int id = blockIdx.x;
  if (id < kb * nb)
    sgd_update_block<T>(id % kb, id / kb, u.W32, u.vW, u.dW, u.N, u.K, u.ldk, (bf16*)u.W16, (T*)u.WT, u.ldn, u.lr, u.mu);
  else
    bias_grad_update_block<T>(id - kb * nb, (const T*)u.dZT, u.ldt, u.N, u.B, u.db, u.b, u.vb, u.lr, u.mu);
}

// ---------------------------------------------------------------------------------
// a layer's float32 matrix and vector between the library's padded rows and a caller's dense ones
// ---------------------------------------------------------------------------------
// One launch instead of a rectangle copy and a plain one by the runtime, each of which costs a small layer more than its step's
// launches (host side: 12 us a copy).
__global__ __launch_bounds__(256) void copy_layer_kernel(const float* __restrict__ W, int lds, float* __restrict__ Wd, int ldd, int N, int K,
                                                         const float* __restrict__ b, float* __restrict__ bd, int vec) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int per = vec ? 4 : 1, cols = (K + per - 1) / per;
  if (W) {
    for (int n = blockIdx.x; n < N; n += gridDim.x)
      for (int c = threadIdx.x; c < cols; c += 256) {
        if (vec) *(f32x4*)(Wd + (size_t)n * ldd + 4 * c) = *(const f32x4*)(W + (size_t)n * lds + 4 * c);
        else Wd[(size_t)n * ldd + c] = W[(size_t)n * lds + c];
      }
  }
  if (b)
    for (int n = blockIdx.x * 256 + threadIdx.x; n < N; n += gridDim.x * 256) bd[n] = b[n];
}

}  // namespace

hipError_t launch_copy_transpose(int dtype, const void* in, int ldin, int R, int C, void* out, int ldo, void* outT,
                                 int ldt, int pad_t, const void* mask, int ldmask, hipStream_t s) {
  dim3 grid((C + 63) / 64, (R + 63) / 64);
  // 16-byte vectors when every row of every operand starts on a 16-byte boundary and the transposed output takes
  // whole row chunks; the element-wise kernel otherwise (a dense caller matrix whose width is not a multiple of V)
  const int V = dtype == 1 ? 8 : 4;
  const int rows_t = pad_t ? ((R + 7) & ~7) : R;
  const bool aligned = ((((uintptr_t)in | (uintptr_t)out | (uintptr_t)outT | (uintptr_t)mask) & 15) == 0) && ldin % V == 0 &&
                       (!out || ldo % V == 0) && (!outT || (ldt % V == 0 && rows_t % V == 0)) && (!mask || ldmask % V == 0);
  if (aligned) {
    // large bf16 matrices: 128 x 128 tiles once they still give every compute unit several workgroups
    if (dtype == 1 && (long)((C + 127) / 128) * ((R + 127) / 128) >= 1024) {
      dim3 grid128((C + 127) / 128, (R + 127) / 128);
      copy_transpose_vec_kernel<bf16, 128><<<grid128, 256, 0, s>>>((const bf16*)in, ldin, R, C, (bf16*)out, ldo, (bf16*)outT, ldt,
                                                                   rows_t, (const bf16*)mask, ldmask);
    } else if (dtype == 1)
      copy_transpose_vec_kernel<bf16, 64><<<grid, 256, 0, s>>>((const bf16*)in, ldin, R, C, (bf16*)out, ldo, (bf16*)outT, ldt, rows_t,
                                                               (const bf16*)mask, ldmask);
    else
      copy_transpose_vec_kernel<float, 64><<<grid, 256, 0, s>>>((const float*)in, ldin, R, C, (float*)out, ldo, (float*)outT, ldt,
                                                                rows_t, (const float*)mask, ldmask);
    return hipGetLastError();
  }
  if (dtype == 1)
    copy_transpose_kernel<bf16><<<grid, 256, 0, s>>>((const bf16*)in, ldin, R, C, (bf16*)out, ldo, (bf16*)outT, ldt, pad_t,
                                                     (const bf16*)mask, ldmask);
  else
    copy_transpose_kernel<float><<<grid, 256, 0, s>>>((const float*)in, ldin, R, C, (float*)out, ldo, (float*)outT, ldt, pad_t,
                                                      (const float*)mask, ldmask);
  return hipGetLastError();
}

int mse_partial_count(int B, int D) { return ((D + 63) / 64) * ((B + 63) / 64); }

hipError_t launch_mse_loss_grad(int dtype, const void* AL, int ld, const int32_t* y, const float* table, int classes,
                                int B, int D, int relu_last, void* dZ, void* dZT, int ldt, float* partials, unsigned* bad_ids,
                                hipStream_t s) {
  dim3 grid((D + 63) / 64, (B + 63) / 64);
  const float scale = (float)(2.0 / ((double)B * (double)D));
  if (dtype == 1)
    mse_loss_grad_kernel<bf16><<<grid, 256, 0, s>>>((const bf16*)AL, ld, y, table, classes, B, D, relu_last, scale, (bf16*)dZ,
                                                    (bf16*)dZT, ldt, partials, bad_ids);
  else
    mse_loss_grad_kernel<float><<<grid, 256, 0, s>>>((const float*)AL, ld, y, table, classes, B, D, relu_last, scale, (float*)dZ,
                                                     (float*)dZT, ldt, partials, bad_ids);
  return hipGetLastError();
}

// Four rows per wavefront in one launch as long as the logits fit into registers and the transposed stores are whole enough.
// A step of 64-C, microseconds, one launch / one row per wavefront and a transpose: float32 256 x 47 15.6 / 18.0, 1024 x 200
// 18.6 / 19.3, 1024 x 256 18.5 / 19.9, 8192 x 47 40.5 / 43.2, 8192 x 256 49.6 / 53.1; bf16 256 x 47 15.5 / 18.0, 1024 x 128 16.4 /
// 18.1, 2048 x 128 17.5 / 17.9, 8192 x 128 26.1 / 26.6, but 256 x 200 18.6 / 18.0, 2048 x 200 22.0 / 18.6, 2048 x 256 21.9 / 18.5.
int xent_launch_count(int dtype, int C) { return C <= (dtype == 1 ? 128 : 256) ? 1 : 2; }

template <typename T>
static hipError_t launch_xent(int dtype, const void* ZL, int ld, const int32_t* y, int B, int C, int relu_last, void* dZ, void* dZT, int ldt,
                              float* partials, unsigned* bad_ids, hipStream_t s) {
  const float inv_b = (float)(1.0 / (double)B);
  constexpr int NC = sizeof(T) == 2 ? 2 : 4;
  if (xent_launch_count(dtype, C) == 1) {
    const int grid = (((B + 7) & ~7) / 4 + 3) / 4;
    if (C <= 64)
      xent_loss_grad_kernel<T, 1><<<grid, 256, 0, s>>>((const T*)ZL, ld, y, B, C, relu_last, inv_b, (T*)dZ, (T*)dZT, ldt, partials, bad_ids);
    else
      xent_loss_grad_kernel<T, NC><<<grid, 256, 0, s>>>((const T*)ZL, ld, y, B, C, relu_last, inv_b, (T*)dZ, (T*)dZT, ldt, partials, bad_ids);
    return hipGetLastError();
  }
  xent_loss_grad_wide_kernel<T><<<(B + 3) / 4, 256, 0, s>>>((const T*)ZL, ld, y, B, C, relu_last, inv_b, (T*)dZ, partials, bad_ids);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess || !dZT ? e : launch_copy_transpose(dtype, dZ, ld, B, C, nullptr, 0, dZT, ldt, 1, nullptr, 0, s);
}

hipError_t launch_xent_loss_grad(int dtype, const void* ZL, int ld, const int32_t* y, int B, int C, int relu_last,
                                 void* dZ, void* dZT, int ldt, float* partials, unsigned* bad_ids, hipStream_t s) {
  return dtype == 1 ? launch_xent<bf16>(dtype, ZL, ld, y, B, C, relu_last, dZ, dZT, ldt, partials, bad_ids, s)
                    : launch_xent<float>(dtype, ZL, ld, y, B, C, relu_last, dZ, dZT, ldt, partials, bad_ids, s);
}

hipError_t launch_hurry(unsigned* hurry, unsigned value, hipStream_t s) {
  hurry_kernel<<<1, 1, 0, s>>>(hurry, value);
  return hipGetLastError();
}

hipError_t launch_copy_layer(const float* W, int lds, float* Wd, int ldd, int N, int K, const float* b, float* bd, hipStream_t s) {
  const int vec = K % 4 == 0 && lds % 4 == 0 && ldd % 4 == 0 && (((uintptr_t)W | (uintptr_t)Wd) & 15) == 0;
  copy_layer_kernel<<<N < 4096 ? N : 4096, 256, 0, s>>>(W, lds, Wd, ldd, N, K, b, bd, vec);
  return hipGetLastError();
}

hipError_t launch_reduce_loss(const float* partials, int n, double scale, float* out0, float* out1, hipStream_t s) {
  reduce_loss_kernel<<<1, 256, 0, s>>>(partials, n, scale, out0, out1);
  return hipGetLastError();
}

hipError_t launch_layer_update(int dtype, float* W32, float* vW, const float* dW, int N, int K, int ldk, void* W16, void* WT,
                               int ldn, const void* dZT, int ldt, int B, float* db, float* b, float* vb, float lr, float mu, hipStream_t s) {
  const LayerUpdate u{W32, vW, dW, N, K, ldk, dtype == 1 ? W16 : nullptr, WT, ldn, dZT, ldt, B, db, b, vb, lr, mu};
  const int grid = ((K + 63) / 64) * ((N + 63) / 64) + (N + 3) / 4;
  if (dtype == 1) layer_update_kernel<bf16><<<grid, 256, 0, s>>>(u);
  else layer_update_kernel<float><<<grid, 256, 0, s>>>(u);
  return hipGetLastError();
}

hipError_t launch_update_beside(int dtype, float* W32, float* vW, const float* dW, int N, int K, int ldk, void* W16, void* WT, int ldn,
                                float lr, float mu, int workgroups, int pause, const unsigned* hurry, hipStream_t s) {
  if (workgroups <= 0 || (pause > 0 && !hurry)) return hipErrorInvalidValue;
  if (dtype == 1)
    sgd_update_strided_kernel<bf16><<<workgroups, 256, 0, s>>>(W32, vW, dW, N, K, ldk, (bf16*)W16, (bf16*)WT, ldn, lr, mu, pause, hurry);
  else
    sgd_update_strided_kernel<float><<<workgroups, 256, 0, s>>>(W32, vW, dW, N, K, ldk, nullptr, (float*)WT, ldn, lr, mu, pause, hurry);
  return hipGetLastError();
}

hipError_t launch_refresh_copies(int dtype, float* W32, int N, int K, int ldk, void* W16, void* WT, int ldn, hipStream_t s) {
  dim3 grid((K + 63) / 64, (N + 63) / 64);
  if (dtype == 1) refresh_copies_kernel<bf16><<<grid, 256, 0, s>>>(W32, N, K, ldk, (bf16*)W16, (bf16*)WT, ldn);
  else refresh_copies_kernel<float><<<grid, 256, 0, s>>>(W32, N, K, ldk, nullptr, (float*)WT, ldn);
  return hipGetLastError();
}

}  // namespace slp
