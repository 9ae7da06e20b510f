// The three dense contractions of a segment step -- forward Z = A W^T (+bias, ReLU),
// data gradient dA = dZ W (masked by the ReLU of the layer below) and weight
// gradient dW = dZ^T A (paper Sec. 2-3: fully connected layers trained by
// backpropagation inside one segment) -- all run through ONE kernel family:
//
//     C[m][n] = sum_k A[m][k] * B[n][k]          ("NT": both operands k-contiguous)
//
// The producers lay their outputs out so that every product is NT: the forward and
// data-gradient epilogues store their result both row-major and transposed, and the
// update kernel keeps a transposed copy of the weights.  That way the inner loop is
// the same, best-case one for all three: 16-byte global loads, 16-byte LDS reads,
// no transposition on the operand path.
//
// gfx950 mapping
//   * bf16: v_mfma_f32_16x16x32_bf16 (16x16 blocks; a register-only loop of it sustains 2000-2100 TFLOP/s under the
//     chip's power limit, the 32x32x16 form 1800-1850); float32: v_mfma_f32_32x32x2_f32, four per 16-byte chunk pair.
//     A k-tile is 128 bytes per row for both types (64 bf16 / 32 float), so loads, LDS layout and addressing
//     are byte-identical for the two types.
//   * global -> LDS directly (buffer_load_dwordx4 ... lds): no staging registers and no ds_write instructions.
//     Out-of-range rows and k-tail chunks read as zero through the buffer resource's range check, so ragged
//     M, N and K need no branches.
//   * LDS rows are 128 bytes and the LDS has 64 banks x 4 bytes: a ds_read_b128 is served 16 lanes at a time,
//     i.e. 16 consecutive rows of one k-chunk.  Physical chunk = chunk ^ ((row >> 1) & 7) spreads those 16 rows
//     over all 64 banks (no conflicts counted).  The hardware writes lane l of an LDS-direct load at
//     base + 16 l, so the swizzle is applied on the global side: each lane fetches the chunk that belongs at its
//     physical position.
//   * big products (256x256 tile, bf16) of long contractions: gemm_nt_long_kernel, 4 wavefronts of 128x128, two LDS stages of 64 KB;
//   * of shorter ones: gemm_nt_big_kernel, 8 wavefronts of 128x64, two LDS stages of 64 KB,
//     the loads of a k-tile issued evenly over the whole k-tile (two barriers per k-tile free the stage piecewise);
//     see the comment on that kernel.
//   * small layers have a kernel of their own (gemm_small.hip);
//   * everything else (float32, 128-wide tiles): gemm_nt_kernel, NW wavefronts in a 2 x NW/2 grid, a wavefront
//     owns a (BM/2) x (BN/(NW/2)) sub-tile; NS LDS stages of (BM+BN) x 128 bytes (two for the 256x256 tile, four
//     for the small ones); one barrier per k-tile, after which the loads of tile k+NS are issued; a k-tile is 4
//     pipeline units, the fragments of unit u+1 are read from LDS while unit u multiplies.
//   * in both kernels the source order "a few LDS reads / loads, a few MFMAs" is pinned with scheduling fences,
//     because the compiler's own schedule serialises LDS latency with the matrix pipe.
//   * epilogue: a lane holds 4 consecutive rows of one output column per accumulator register quad, which
//     is one vector store into the transposed output; for the row-major output the quad of lanes holding
//     4 adjacent columns transposes its 4x4 block with DPP moves, after which a lane holds 4 consecutive
//     columns of one row: one vector store as well (2 stores per quad instead of 5).
//     The bf16 outputs of the forward product and the data gradient go through LDS instead and leave as whole 128- and
//     256-byte row segments (see the epilogues).
//   * workgroup -> tile: consecutive workgroup ids go round-robin over the 8 XCDs, so
//     ids are first regrouped per XCD (each XCD gets a contiguous range of tiles and
//     its own 4 MB L2 sees a compact set of operand rows), then walked in column-major groups of 8 tile-rows.
//     Big products whose tile grid divides into 16 x 16 regions are walked region by region instead, all 8 XCDs
//     inside one region at a time (see the kernel).
#include "gemm_device.h"

#include <type_traits>
#include <utility>

namespace slp {
namespace {

constexpr int kGroupM = 8;
constexpr int kRegionWalk = -1;   // GemmArgs::group_m value: walk 16 x 16 regions of tiles (big kernel only)

// The optimiser step in the epilogue of the weight gradient (EPI_WGRAD_UPDATE), one accumulator register quad: the float32
// weights and momenta of 4 consecutive columns of the output row the lane holds after the transpose ...
__device__ __forceinline__ void request_update(const GemmArgs& g, int n, int mb, int lane, f32x4& w, f32x4& vel) {
  const int row = mb + (lane & 3), nb = n - (lane & 3);
  if (row < g.M && nb < g.N) {
    const size_t idx = (size_t)row * g.ldc + nb;
    w = *(const f32x4*)(g.uW + idx);
    if (g.mu != 0.0f) vel = *(const f32x4*)(g.uV + idx);
  }
}
// A lane whose column is past N has a zero row of one operand times the other, which is NaN where that one holds an infinity: the pads of
// gradients, weights and momenta stay zero, whatever a batch holds.
__device__ __forceinline__ void clear_past(const GemmArgs& g, int n, float (&v)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (n >= g.N) v[e] = 0.0f;
}
// ... and the step itself (pad columns hold zeros in every stream and stay zero); then back through the transpose, so that the
// lane holds 4 consecutive output rows of one input column: one vector store into the transposed copy.
template <typename T>
__device__ __forceinline__ void update_quad(const GemmArgs& g, int n, int mb, float (&v)[4], int lane, const f32x4& wo, const f32x4& vo) {
  clear_past(g, n, v);
  quad_transpose(v, lane);
  const int row = mb + (lane & 3), nb = n - (lane & 3);
  float w[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (row < g.M && nb < g.N) {
    const size_t idx = (size_t)row * g.ldc + nb;
    f32x4 vel = f32x4{v[0], v[1], v[2], v[3]};
    if (g.mu != 0.0f) {
      vel = g.mu * vo + vel;
      *(f32x4*)(g.uV + idx) = vel;
    }
    const f32x4 wn = wo - g.lr * vel;
    *(f32x4*)(g.uW + idx) = wn;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = wn[e];
    if (g.uW16) {
      bf16x4 h;
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = (bf16)w[e];
      *(bf16x4*)((bf16*)g.uW16 + idx) = h;
    }
  }
  if (g.uWT) {      // (uniform over the launch)
    quad_transpose(w, lane);
    if (n < g.N && mb < g.M) {     // rows past M inside the vector carry zeros: the pads of the copy stay zero
      typename Vec4<T>::type o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (T)w[e];
      *(typename Vec4<T>::type*)((T*)g.uWT + (size_t)n * g.ldwt + mb) = o;
    }
  }
}

// Epilogue of one accumulator register quad: rows mb..mb+3 of output column n, v[e] = row mb+e.  The 4 lanes of
// a quad hold 4 consecutive columns (n - lane%4 is a multiple of 4), and a lane whose column is past N takes part
// with zeros: nothing here may diverge inside a quad before the transpose.
//   EPI_FWD  : + bias (the caller passes 0 for a column past N), optional ReLU;
//   EPI_DGRAD: zero where the mask (stored transposed) is not positive;
//   both store transposed CT in T as one vector per lane (4 rows of its column; rows past M up to the next
//   multiple of 8 are written as zero) and row-major C after a 4x4 transpose inside the quad, so that a lane
//   stores 4 consecutive columns of one row as one vector (pad columns up to the leading dimension receive
//   zeros);  EPI_WGRAD: float32 row-major, same transposed vector store.
template <typename T, int EPI>
__device__ __forceinline__ void finish_values(const GemmArgs& g, int n, int mb, float bias, float (&v)[4]) {
  if (EPI == EPI_FWD) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] += bias;
      if (g.relu) v[e] = fmaxf(v[e], 0.0f);
    }
  } else if (g.maskT && n < g.N && mb < ((g.M + 7) & ~7)) {     // no mask: the gradient w.r.t. the segment input
    typedef typename Vec4<T>::type mvec_t;
    const mvec_t mk = *(const mvec_t*)((const T*)g.maskT + (size_t)n * g.ldmask + mb);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (!((float)mk[e] > 0.0f)) v[e] = 0.0f;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (mb + e >= g.M || n >= g.N) v[e] = 0.0f;
}
template <typename T, int EPI>
__device__ __forceinline__ void store_quad(const GemmArgs& g, int n, int mb, float bias, float (&v)[4], int lane) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  const bool col_ok = n < g.N;
  const int row = mb + (lane & 3), nb = n - (lane & 3);      // after the transpose: this lane's row, first of its 4 columns
  if (EPI == EPI_WGRAD) {
    clear_past(g, n, v);
    quad_transpose(v, lane);
    if (row < g.M && nb < g.N) *(f32x4_t*)(g.Cf + (size_t)row * g.ldc + nb) = f32x4_t{v[0], v[1], v[2], v[3]};
    return;
  }
  if (EPI == EPI_WGRAD_UPDATE) {
    f32x4 w, vel;
    request_update(g, n, mb, lane, w, vel);
    update_quad<T>(g, n, mb, v, lane, w, vel);
    return;
  }
  if (mb >= ((g.M + 7) & ~7)) return;       // the same for the whole quad
  finish_values<T, EPI>(g, n, mb, bias, v);
  if (g.CT && col_ok) {
    typename Vec4<T>::type o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (T)v[e];
    *(typename Vec4<T>::type*)((T*)g.CT + (size_t)n * g.ldct + mb) = o;
  }
  if (g.C) {
    quad_transpose(v, lane);
    if (row < g.M && nb < g.N) {
      typename Vec4<T>::type o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (T)v[e];
      *(typename Vec4<T>::type*)((T*)g.C + (size_t)row * g.ldc + nb) = o;
    }
  }
}

template <typename T, int BM, int BN, int EPI, int NW, int NS>
__global__ __launch_bounds__(NW * 64) void gemm_nt_kernel(const GemmArgs g) {
#if defined(__HIP_DEVICE_COMPILE__)   // LDS-direct builtins exist in the device pass only; the host pass needs just the launch stub
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int ES = sizeof(T);
  constexpr int CH = Chunk<T>::elems;        // elements per 16-byte chunk
  constexpr int BK = 128 / ES;               // k elements per tile
  constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, STAGE = A_BYTES + B_BYTES;
  constexpr int RPL = 8 * NW;                  // tile rows covered by one load instruction of the whole workgroup
  constexpr int LA = BM / RPL, LB = BN / RPL;  // 16-byte loads per thread per k-tile
  typedef Mma<T> MM;
  constexpr int MB = MM::MB, AH = MM::AH;
  constexpr int CPS = 64 / MB;                 // 16-byte chunks per row that one k-sub-step consumes
  constexpr int KSUB = 8 / CPS;                // k-sub-steps per k-tile
  constexpr int UNITS = KSUB * AH;             // pipeline units per k-tile
  constexpr int WTM = BM / 2, WTN = BN / (NW / 2), MI = WTM / MB, NI = WTN / MB, MIH = MI / AH;
  static_assert(MI % AH == 0 && UNITS % 2 == 0 && KSUB % 2 == 0, "buffer parity must repeat from tile to tile");

  // ---- workgroup -> tile ------------------------------------------------------------
  const int tilesM = (g.M + BM - 1) / BM, tilesN = (g.N + BN - 1) / BN;
  const int total = tilesM * tilesN;
  int tid;
  {
    const int pid = blockIdx.x, xcd = pid % kXcds, q = pid / kXcds;
    const int base = total / kXcds, rem = total % kXcds;
    tid = xcd * base + (xcd < rem ? xcd : rem) + q;
  }
  const int group_m = g.group_m > 0 ? g.group_m : kGroupM;
  const int width = group_m * tilesN;
  const int group = tid / width, first_m = group * group_m;
  const int gsz = (tilesM - first_m) < group_m ? (tilesM - first_m) : group_m;
  const int tm = first_m + (tid % width) % gsz, tn = (tid % width) / gsz;
  const int m0 = tm * BM, n0 = tn * BN;

  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wm = w & 1, wn = w >> 1;
  const int lgrp = lane / MB, lrow = lane % MB;

  // ---- global load addressing --------------------------------------------------------
  const int Kr = (g.K + CH - 1) / CH * CH;   // chunk-granular contraction length
  const __amdgpu_buffer_rsrc_t rsrcA =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.A), 0, (int)((size_t)g.M * g.lda * ES), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcB =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.B), 0, (int)((size_t)g.N * g.ldb * ES), 0x00020000);
  // Direct-to-LDS loads: load i of wavefront w fills LDS rows [8w + RPL i, 8w + RPL i + 8) of the tile
  // (RPL = 8 x wavefronts), lane l writing 16 bytes at (row 8w + RPL i + l/8, physical chunk l%8) --
  // the hardware places lane l at base + 16*l.  The XOR swizzle is therefore applied on the global
  // side: the lane fetches the logical chunk that belongs at its physical position.
  const int prow = w * 8 + (lane >> 3);                   // + RPL i
  const int pchunk = (lane & 7) ^ ((prow >> 1) & 7);      // logical k-chunk fetched by this lane
  uint32_t voffA[LA], voffB[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) voffA[i] = (uint32_t)(((size_t)(m0 + prow + RPL * i) * g.lda + pchunk * CH) * ES);
#pragma unroll
  for (int i = 0; i < LB; ++i) voffB[i] = (uint32_t)(((size_t)(n0 + prow + RPL * i) * g.ldb + pchunk * CH) * ES);
  typedef __attribute__((address_space(3))) void* lds_ptr_t;
  const uint32_t lds_wave = (uint32_t)__builtin_amdgcn_readfirstlane(w * 8 * 128);
  const int kc = pchunk;

  // ---- fragment addressing -------------------------------------------------------------
  const uint32_t fragA = (uint32_t)((wm * WTM + lrow) * 128);
  const uint32_t fragB = (uint32_t)(A_BYTES + (wn * WTN + lrow) * 128);
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

  // Pipeline unit u of a k-tile = k-sub-step u / AH, part u % AH of the wavefront's rows: MIH A fragments (buffer u & 1)
  // against the sub-step's NI B fragments (buffer (u / AH) & 1, read together with part 0).
  u32x4 af[2][MIH], bfr[2][NI];
  // Every k-sub-step is written out as small groups "a few loads/stores + a few MFMAs",
  // fenced so that the compiler keeps the interleaving: the matrix pipe always has work
  // queued while LDS and global traffic for later sub-steps is in flight.
  constexpr int NRD = MIH + NI;                              // most fragment reads any unit needs (those with part 0)
  constexpr int NLD = LA + LB;                               // global loads / LDS writes per k-tile
  constexpr int NMM = MIH * NI;                              // MFMA groups per unit
  auto reads_of = [](int u) { return MIH + (u % AH == 0 ? NI : 0); };
  auto read_one = [&](int stage, int u, int r) {             // read r of the fragments unit u multiplies
    const unsigned char* sb = smem + stage * STAGE;
    const int kk = u / AH, h = u % AH;
    if (r < MIH) af[u & 1][r] = *(const u32x4*)(sb + fragA + (h * MIH + r) * MB * 128 + xo[kk]);
    else bfr[kk & 1][r - MIH] = *(const u32x4*)(sb + fragB + (r - MIH) * MB * 128 + xo[kk]);
  };
  auto mma_one = [&](int u, int m) {
    MM::mma(acc[(u % AH) * MIH + m / NI][m % NI], af[u & 1][m / NI], bfr[(u / AH) & 1][m % NI]);
  };
  auto gload_one = [&](int kt, int stage, int i) {
    const bool in_k = kt * BK + kc * CH < Kr;      // past the end of K every load becomes a zero fill
    const uint32_t koff = (uint32_t)kt * 128u;
    if (i < LA)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcA, (lds_ptr_t)(smem + stage * STAGE + lds_wave + i * RPL * 128), 16,
                                               in_k ? voffA[i] + koff : kOutOfRange, 0, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB, (lds_ptr_t)(smem + stage * STAGE + A_BYTES + lds_wave + (i - LA) * RPL * 128), 16,
                                               in_k ? voffB[i - LA] + koff : kOutOfRange, 0, 0, 0);
  };
// s_waitcnt immediate: wait until at most n vector-memory operations are outstanding (other counters untouched)
#define VMCNT(n) ((((n) & 15) | 0x0F70 | (((n) >> 4) << 14)))
#define SLP_FENCE() __builtin_amdgcn_sched_barrier(0)

  const int nk = (Kr + BK - 1) / BK;
#pragma unroll
  for (int st = 0; st < NS; ++st)
#pragma unroll
    for (int i = 0; i < NLD; ++i) gload_one(st, st, i);
  SLP_FENCE();
  // what the epilogue of bf16 outputs reads, behind the first operands
  constexpr bool kStaged = ES == 2 && (EPI == EPI_FWD || EPI == EPI_DGRAD);
  float bias[NI];
  uint32_t bits[NI];                     // data gradient: this lane's rows of the mask, bit 4 i + e (GemmArgs::bits)
  if constexpr (kStaged) {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int n = n0 + wn * WTN + j * MB + lrow;
      bias[j] = 0.0f;
      bits[j] = 0;
      if (EPI == EPI_FWD && n < g.N) bias[j] = g.bias[n];
      if (EPI == EPI_DGRAD && g.bits && n < g.N && m0 + wm * WTM < g.M)
        bits[j] = ((const uint16_t*)(g.bits + (size_t)n * g.ldbits + (m0 >> 5) + lgrp))[wm];
    }
    SLP_FENCE();
  }
  __builtin_amdgcn_s_waitcnt(VMCNT((NS - 1) * NLD));
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NRD; ++r) read_one(0, 0, r);
  auto rd_lo = [](int g, int n) { return 2 * g < n ? 2 * g : n; };
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt % NS, nxt = (kt + 1) % NS;
#pragma unroll
    for (int u = 0; u < UNITS - 1; ++u) {
#pragma unroll
      for (int g = 0; g < NRD; ++g) {
#pragma unroll
        for (int r = rd_lo(g, reads_of(u + 1)); r < rd_lo(g + 1, reads_of(u + 1)); ++r) read_one(cur, u + 1, r);
#pragma unroll
        for (int m = g * NMM / NRD; m < (g + 1) * NMM / NRD; ++m) mma_one(u, m);
        SLP_FENCE();
      }
    }
    // tile kt+1 must have landed in stage nxt (this wave's part), and every wave must be done reading stage cur
    if (NS == 2) {
      __builtin_amdgcn_s_waitcnt(VMCNT(0));
      __syncthreads();
    } else {
      // tiles kt+2 .. kt+NS-1 stay in flight.  A bare barrier between compiler fences: the workgroup release fence
      // of __syncthreads() waits for EVERY outstanding LDS-direct load.  What the barrier has to order is waited for
      // by hand: this wavefront's loads of tile kt+1 (vmcnt) and its LDS reads of stage cur (lgkmcnt 0).
      __builtin_amdgcn_s_waitcnt(VMCNT((NS - 2) * NLD) & 0xF0FF);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int g = 0; g < NRD; ++g) {
#pragma unroll
      for (int r = rd_lo(g, NRD); r < rd_lo(g + 1, NRD); ++r) read_one(nxt, 0, r);
#pragma unroll
      for (int i = g * NLD / NRD; i < (g + 1) * NLD / NRD; ++i) gload_one(kt + NS, cur, i);
#pragma unroll
      for (int m = g * NMM / NRD; m < (g + 1) * NMM / NRD; ++m) mma_one(UNITS - 1, m);
      SLP_FENCE();
    }
  }
  __builtin_amdgcn_s_waitcnt(VMCNT(0));
#undef SLP_FENCE

  // ---- epilogue ----------------------------------------------------------------------------
  // Accumulator layout of an MB x MB block: lane holds column n = lane % MB and, in register r, row
  // (64 / MB * 4) * (r / 4) + 4 * (lane / MB) + (r % 4): four consecutive rows per register quad, which is what
  // makes the transposed store a vector store.
  constexpr int NQ = MM::ACC / 4;
  if constexpr (EPI == EPI_WGRAD_UPDATE) {
    // The weights and momenta of all blocks (4 wavefronts: of one row of blocks, the registers of two workgroups per compute
    // unit do not hold more) are requested before any of them is used: quad by quad every load waited for the stores of the
    // quad before (loads and stores share one counter).  8 wavefronts, all blocks against a row of blocks at a time, buffers
    // not in cache: 4096x784x1024 bf16 24.0 -> 23.2 us, 2048x4096x1024 65 -> 55, float32 2048x2048x256 32.5 -> 31.5.
    constexpr int IB = NW == 8 && MI * NI * NQ * 8 <= 128 ? MI : 1;
#pragma unroll
    for (int i0 = 0; i0 < MI; i0 += IB) {
      f32x4 w[IB][NI][NQ], v[IB][NI][NQ];
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            request_update(g, n0 + wn * WTN + j * MB + lrow, m0 + wm * WTM + (i0 + i) * MB + (256 / MB) * q + 4 * lgrp, lane, w[i][j][q], v[i][j][q]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = acc[i0 + i][j][4 * q + e];
            update_quad<T>(g, n0 + wn * WTN + j * MB + lrow, m0 + wm * WTM + (i0 + i) * MB + (256 / MB) * q + 4 * lgrp, x, lane, w[i][j][q], v[i][j][q]);
            __builtin_amdgcn_sched_barrier(0);
          }
    }
    return;
  }
  typedef typename Vec4<T>::type vec4;
  if constexpr (kStaged) {
    // bf16: straight from the accumulators a store covers 32 bytes of each of 16 rows.  The tile goes through LDS in both layouts, rows
    // of 256 bytes transposed and 2 BN row-major (no bank conflicts on either side), and leaves in 16-byte pieces of whole row segments.
    // Forward, microseconds before / after: 1024x4096, K = 64 9.2 / 8.3, 784 15.7 / 14.7, 4096 36.8 / 35.5, 2048x4096x1024 26.2 / 23.3,
    // 1024x2048x4096 26.7 / 25.0, 1280x1664x1024 13.8 / 12.7.  (float32 blocks are 32 columns: whole lines already.)
    // The mask of the data gradient comes as bits; as 8-byte pieces of the activation behind the stores it cost 5 us on 2048x4096, all of
    // them requested before the k-loop 1 us more than that at K = 4096.
    constexpr int CROW = BN * 2, CCH = CROW / 16, TCH = BM / 8;
    static_assert(BM == 128 && WTM == 64 && BN * 256 + BM * CROW <= NS * STAGE, "half a word of mask bits per lane; both layouts fit into the stages");
    unsigned char *const ct = smem, *const cm = smem + BN * 256;
    auto at_t = [&](int r, int c) { return ct + r * 256 + ((c ^ (r & 15)) << 4); };
    auto at_m = [&](int r, int c) { return cm + r * CROW + ((c ^ (CCH == 16 ? (r << 1) & 14 : r & 6)) << 4); };
    __syncthreads();                     // nobody reads the stages any more and every load into them has landed
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int nl = wn * WTN + j * MB + lrow, n = n0 + nl;
      uint32_t word = 0;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int ml = wm * WTM + i * MB + 4 * lgrp;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][e];
        if (EPI == EPI_DGRAD && g.bits) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (!((bits[j] >> (4 * i + e)) & 1u) || n >= g.N || m0 + ml + e >= g.M) v[e] = 0.0f;
        } else {
          finish_values<T, EPI>(g, n, m0 + ml, bias[j], v);
        }
        if (EPI == EPI_FWD) {
#pragma unroll
          for (int e = 0; e < 4; ++e) word |= (uint32_t)((float)(T)v[e] > 0.0f) << (4 * i + e);
        }
        if (g.CT) *(vec4*)(at_t(nl, ml >> 3) + (ml & 4) * 2) = vec4{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
        if (g.C) {
          quad_transpose(v, lane);
          const int nb = nl - (lane & 3);
          *(vec4*)(at_m(ml + (lane & 3), nb >> 3) + (nb & 4) * 2) = vec4{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
        }
      }
      if (EPI == EPI_FWD && g.bits_out && n < g.N && m0 + wm * WTM < g.M)
        ((uint16_t*)(g.bits_out + (size_t)n * g.ldbits + (m0 >> 5) + lgrp))[wm] = (uint16_t)word;
    }
    __syncthreads();
    if (g.CT) {
#pragma unroll
      for (int x = t; x < BN * TCH; x += NW * 64) {
        const int r = x / TCH, c = x % TCH;
        if (n0 + r < g.N && m0 + c * 8 < g.M) *(u32x4*)((T*)g.CT + (size_t)(n0 + r) * g.ldct + m0 + c * 8) = *(const u32x4*)at_t(r, c);
      }
    }
    if (g.C) {
#pragma unroll
      for (int x = t; x < BM * CCH; x += NW * 64) {
        const int r = x / CCH, c = x % CCH;
        if (m0 + r < g.M && n0 + c * 8 < g.N) *(u32x4*)((T*)g.C + (size_t)(m0 + r) * g.ldc + n0 + c * 8) = *(const u32x4*)at_m(r, c);
      }
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int n = n0 + wn * WTN + j * MB + lrow;
    float bias = 0.0f;
    if (EPI == EPI_FWD && n < g.N) bias = g.bias[n];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int q = 0; q < MM::ACC / 4; ++q) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * q + e];
        store_quad<T, EPI>(g, n, m0 + wm * WTM + i * MB + (256 / MB) * q + 4 * lgrp, bias, v, lane);
        // keep the scheduler from hoisting every block's address arithmetic and mask
        // loads to the top of the epilogue (that spills registers)
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
#endif
}

// workgroup -> 256x256 tile
__device__ __forceinline__ void big_tile(const GemmArgs& g, int& tm, int& tn) {
  const int tilesM = (g.M + 255) / 256, tilesN = (g.N + 255) / 256;
  const int pid = blockIdx.x, xcd = pid % kXcds, q = pid / kXcds;
  if (g.group_m == kRegionWalk) {
    // All 8 XCDs work on one 16 x 16 region of tiles at a time, as 2 x 4 blocks of 8 x 4 tiles (one block per XCD,
    // one tile per compute unit): 32 operand strips feed 256 concurrent tiles, and what one XCD fetched is in the
    // memory-side cache for the XCDs that share its strips.  Regions are walked down the rows first.
    const int r = q / 32, sl = q % 32, regM = tilesM / 16;
    tm = (r % regM) * 16 + (xcd % 2) * 8 + sl % 8;
    tn = (r / regM) * 16 + (xcd / 2) * 4 + sl / 8;
    return;
  }
  const int total = tilesM * tilesN, base = total / kXcds, rem = total % kXcds;
  const int tid = xcd * base + (xcd < rem ? xcd : rem) + q;
  const int group_m = g.group_m > 0 ? g.group_m : kGroupM;
  const int width = group_m * tilesN;
  const int group = tid / width, first_m = group * group_m;
  const int gsz = (tilesM - first_m) < group_m ? (tilesM - first_m) : group_m;
  tm = first_m + (tid % width) % gsz;
  tn = (tid % width) / gsz;
}

// Big bf16 products of shorter contractions: 256x256 tile, 8 wavefronts in a 2 x 4 grid, 128 x 64 each,
// v_mfma_f32_16x16x32_bf16, two LDS stages of 64 KB.
// A k-tile (64 k) is 4 units: (row half h, k-sub-step kk) in the order (0,0) (0,1) (1,0) (1,1), each 4 A fragments
// against the NB B fragments of the sub-step.  The B fragments of a k-tile stay in registers for the whole tile, the A
// fragments are read one unit ahead.  That order frees LDS early: after unit 0 nothing of this stage's B rows and h=0
// A rows is needed any more, after unit 2 the h=1 A rows are free too.  Two barriers per k-tile (X after unit 0, Y
// after unit 2) let the LDS-direct loads of tile kt+2 be issued evenly over the whole k-tile, a quarter of them per
// unit.  Issued in one burst after a single barrier (as gemm_nt_kernel does) they cost the unit that issues them 3x its
// MFMA time: measured per unit with the cycle counter, 570 / 581 / 498 / 1578 cycles against 512 of MFMAs each.
// Sustained on 8192x16384x16384: 1295-1315 -> 1365-1415 TFLOP/s.
// Register budget: 216-222 per lane (allocated as 224), two wavefronts per SIMD; the 64 that remain of the SIMD's 512
// are what the weight-update kernel running beside the products is held to -- above 224 here it no longer fits.
template <int EPI, int NW>
__global__ __launch_bounds__(NW * 64) void gemm_nt_big_kernel(const GemmArgs g) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef bf16 T;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // highest wave priority: on a compute unit shared with an update workgroup the product's loads are issued first
  // (+0.4 % per step on the comparison configuration; no effect when the kernel runs alone)
  __builtin_amdgcn_s_setprio(3);
  constexpr int BM = 256, BN = 256, ES = 2, CH = 8, BK = 64;
  constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
  static_assert(NW == 8, "loads, schedule and epilogue are laid out for 8 wavefronts of 128 x 64");
  constexpr int WN = NW / 2;             // wavefront columns
  constexpr int WTN = BN / WN;           // columns per wavefront
  constexpr int NB = WTN / 16;           // B fragments per sub-step
  constexpr int RPL = 8 * NW;            // rows one load instruction of the workgroup covers
  constexpr int NBLK = 256 / RPL;        // row blocks (= loads per lane) per operand per k-tile
  constexpr int NL = 2 * NBLK;           // loads per lane per k-tile
  constexpr int LPU = NL / 4;            // loads per unit
  constexpr int NSLOT = 2 * NB;          // slots of 2 MFMAs per unit

  int tm, tn;
  big_tile(g, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;

  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wm = w & 1, wn = w >> 1;
  const int lgrp = lane >> 4, lrow = lane & 15;

  const int Kr = (g.K + CH - 1) / CH * CH;
  const __amdgpu_buffer_rsrc_t rsrcA =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.A), 0, (int)((size_t)g.M * g.lda * ES), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcB =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.B), 0, (int)((size_t)g.N * g.ldb * ES), 0x00020000);
  // load i of the workgroup fills rows [RPL i, RPL i + RPL) of an operand's 256; wavefront w rows 8w..8w+7 of those
  const int prow = w * 8 + (lane >> 3);
  const int pchunk = (lane & 7) ^ ((prow >> 1) & 7);
  uint32_t voffA[NBLK], voffB[NBLK];
#pragma unroll
  for (int i = 0; i < NBLK; ++i) voffA[i] = (uint32_t)(((size_t)(m0 + prow + RPL * i) * g.lda + pchunk * CH) * ES);
#pragma unroll
  for (int i = 0; i < NBLK; ++i) voffB[i] = (uint32_t)(((size_t)(n0 + prow + RPL * i) * g.ldb + pchunk * CH) * ES);
  typedef __attribute__((address_space(3))) void* lds_ptr_t;
  const uint32_t lds_wave = (uint32_t)__builtin_amdgcn_readfirstlane(w * 8 * 128);
  const int kc = pchunk;

  const uint32_t fragA = (uint32_t)((wm * 128 + lrow) * 128);
  const uint32_t fragB = (uint32_t)(A_BYTES + (wn * WTN + lrow) * 128);
  uint32_t xo[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) xo[kk] = (uint32_t)(((kk * 4 + lgrp) ^ ((lane >> 1) & 7)) << 4);

  f32x4 acc[8][NB];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

  u32x4 af[2][4], bfr[2][NB];
  // The NL loads of a k-tile in issue order: first the 3/4 that fill the rows free after unit 0 (A rows of half h = 0 of
  // both wavefront rows, all B rows), then the A rows of half h = 1.  Entry < NBLK: A row block, else B row block.
  auto gload = [&](int kt, int stage, int idx) {
    const bool in_k = kt * BK + kc * CH < Kr;
    const uint32_t koff = (uint32_t)kt * 128u;
    constexpr int order[8] = {0, 4, 2, 5, 6, 7, 1, 3};
    const int o = order[idx];
    if (o < NBLK)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcA, (lds_ptr_t)(smem + stage * STAGE + lds_wave + o * RPL * 128), 16,
                                               in_k ? voffA[o] + koff : kOutOfRange, 0, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB, (lds_ptr_t)(smem + stage * STAGE + A_BYTES + lds_wave + (o - NBLK) * RPL * 128), 16,
                                               in_k ? voffB[o - NBLK] + koff : kOutOfRange, 0, 0, 0);
  };
  auto read_a = [&](int stage, int h, int kk, int buf, int r) {
    af[buf][r] = *(const u32x4*)(smem + stage * STAGE + fragA + (h * 4 + r) * 16 * 128 + xo[kk]);
  };
  auto read_b = [&](int stage, int kk, int c) {
    bfr[kk][c] = *(const u32x4*)(smem + stage * STAGE + fragB + c * 16 * 128 + xo[kk]);
  };
  // m = 0..4 NB - 1: A fragment ia = m / NB against the B fragments in turn, forwards for even ia and backwards for
  // odd ia, so that from one MFMA to the next only one of the two operands changes.  The chip is power-limited under
  // this load and operand lines that do not toggle cost less: measured +0.8 % on 8192x16384x16384 and 16384x16384x8192
  // against walking the B fragments forwards every time (three alternating runs each, spread 0.1 %).
  auto mma = [&](int h, int kk, int buf, int m) {
    const int ia = m / NB, ib = (ia & 1) ? NB - 1 - m % NB : m % NB;
    acc[h * 4 + ia][ib] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
        __builtin_bit_cast(bf16x8, af[buf][ia]), __builtin_bit_cast(bf16x8, bfr[kk][ib]), acc[h * 4 + ia][ib], 0, 0, 0);
  };
#define VMCNT(n) ((((n) & 15) | 0x0F70 | (((n) >> 4) << 14)))
#define SLP_FENCE() __builtin_amdgcn_sched_barrier(0)
#define SLP_BARRIER(n)                                              \
  do {                                                              \
    __builtin_amdgcn_s_waitcnt(VMCNT(n) & 0xF0FF);                  \
    asm volatile("" ::: "memory");                                  \
    __builtin_amdgcn_s_barrier();                                   \
    asm volatile("" ::: "memory");                                  \
  } while (0)

  const int nk = (Kr + BK - 1) / BK;
  // A slot = up to two memory operations followed by 2 MFMAs.  Operation codes: 0 none, 1 + r: read A fragment r,
  // 5 + c: read B fragment c, 13 + i: the unit's load i.  Reads are ordered by first use in the next unit (A0, B0.., A1..).
  struct Slot { int a, b; };
  // the reads go first (they have then returned when the unit ends in a barrier: +1 % over reads
  // spread through the unit), the loads after them
  constexpr Slot kWide[8] = {{1, 5}, {6, 7}, {8, 2}, {3, 4}, {13, 0}, {0, 0}, {14, 0}, {0, 0}};
  constexpr Slot kNarrow[8] = {{1, 2}, {3, 4}, {13, 0}, {0, 0}, {0, 0}, {14, 0}, {0, 0}, {0, 0}};
  // one unit: fragments of (h, kk) from af[buf], bfr[kk]; reads for the next unit (A fragments of (rh, rk) into
  // af[buf ^ 1], and, in a wide unit, the B fragments of sub-step rk) from stage rs; loads lbase.. of tile lkt into stage ls
  auto unit = [&](bool wide, int h, int kk, int buf, int rs, int rh, int rk, int lkt, int ls, int lbase) {
#pragma unroll
    for (int sl = 0; sl < NSLOT; ++sl) {
      const Slot so = wide ? kWide[sl] : kNarrow[sl];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int op = q == 0 ? so.a : so.b;
        if (op >= 1 && op <= 4) read_a(rs, rh, rk, buf ^ 1, op - 1);
        else if (op >= 5 && op <= 12) read_b(rs, rk, op - 5);
        else if (op >= 13) gload(lkt, ls, lbase + op - 13);
      }
      mma(h, kk, buf, 2 * sl); mma(h, kk, buf, 2 * sl + 1);
      SLP_FENCE();
    }
  };
  // prologue: tile 0 completely and the first 3/4 of the loads of tile 1
#pragma unroll
  for (int i = 0; i < NL; ++i) gload(0, 0, i);
#pragma unroll
  for (int i = 0; i < 3 * LPU; ++i) gload(1, 1, i);
  SLP_BARRIER(3 * LPU);
#pragma unroll
  for (int r = 0; r < 4; ++r) read_a(0, 0, 0, 0, r);
#pragma unroll
  for (int c = 0; c < NB; ++c) read_b(0, 0, c);

  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1, nxt = cur ^ 1;
    unit(true, 0, 0, 0, cur, 0, 1, kt + 1, nxt, 3 * LPU);     // reads A(0,1), B(1); last quarter of tile kt+1's loads
    SLP_BARRIER(4 * LPU);   // X: this tile's h=1 A rows have landed; nobody reads B / h=0 A rows of stage cur any more
    unit(false, 0, 1, 1, cur, 1, 0, kt + 2, cur, 0);          // reads A(1,0); first quarter of tile kt+2's loads
    unit(false, 1, 0, 0, cur, 1, 1, kt + 2, cur, LPU);        // reads A(1,1); second quarter
    SLP_BARRIER(3 * LPU);   // Y: B and h=0 A rows of tile kt+1 have landed in stage nxt; h=1 A rows of stage cur are free
    unit(true, 1, 1, 1, nxt, 0, 0, kt + 2, cur, 2 * LPU);     // reads next tile's A(0,0), B(0); third quarter
  }
  __builtin_amdgcn_s_waitcnt(VMCNT(0));
#undef SLP_FENCE
#undef SLP_BARRIER
#undef VMCNT

  if constexpr (EPI == EPI_WGRAD || EPI == EPI_WGRAD_UPDATE) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int n = n0 + wn * WTN + j * 16 + lrow;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][e];
        store_quad<T, EPI>(g, n, m0 + wm * 128 + i * 16 + 4 * lgrp, 0.0f, v, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    // Forward / data gradient: both outputs are bf16, and an accumulator block holds only 32 contiguous bytes of an
    // output row (or column).  Each wavefront therefore stages its own 128 x 64 sub-tile through a private 16 KB
    // region of the (now free) LDS stages, once transposed (64 rows of 256 bytes) and once row-major (128 rows of 128
    // bytes), and stores it as whole row segments in 16-byte pieces per lane: full cache lines on both sides, and no
    // workgroup barrier after the first one (LDS operations of one wavefront execute in order).  16-byte chunk c of
    // a staged row r sits at chunk c ^ (r & 15) (transposed) / c ^ ((r >> 1) & 7) (row-major), which keeps the
    // 8-byte writes and the 16-byte reads of a wavefront free of bank conflicts.
    // The data gradient's ReLU mask comes as bits (GemmArgs::bits, from the forward product of the layer below, which ran on this tile
    // too): one dword per lane and 16-column block, 4 loads instead of 32 gathered 8-byte pieces of the
    // transposed activation (the gather was 10 of the epilogue's 17 us per tile).  Applying the bf16 mask on the way out instead, from
    // coalesced 16-byte loads of both layouts of the activation, measured 2-3 % slower on short contractions.  Against one shared 256 x 512-byte
    // staging area with a workgroup barrier around each pass: 8192 x 16384 products -4 % at K = 1024, -0.5 % at K = 16384.
    typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
    const int rowW = m0 + wm * 128, colW = n0 + wn * WTN;     // origin of this wavefront's sub-tile
    // data gradient with the mask as bits: the 32 bits a lane needs per accumulator column are one dword
    uint32_t mbits[NB];
    if (EPI == EPI_DGRAD && g.bits) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int n = colW + j * 16 + lrow;
        mbits[j] = (n < g.N && rowW < g.M) ? g.bits[(size_t)n * g.ldbits + (rowW >> 5) + lgrp] : 0u;   // rowW >= M: no such block in the row
      }
    }
    __syncthreads();   // every wavefront's (zero-fill) loads have landed and its fragment reads are over
    unsigned char* reg = smem + w * 16384;
    const int Mr = (g.M + 7) & ~7;
    // finish the values in place: bias + ReLU, zeros outside the matrix
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int n = colW + j * 16 + lrow;
      const bool col_ok = n < g.N;
      float bias = 0.0f;
      if (EPI == EPI_FWD && col_ok) bias = g.bias[n];
      uint32_t word = 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int mb = rowW + i * 16 + 4 * lgrp;
        if (EPI == EPI_FWD) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[i][j][e] += bias;
            if (g.relu) acc[i][j][e] = fmaxf(acc[i][j][e], 0.0f);
          }
        } else if (g.bits) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (!((mbits[j] >> (4 * i + e)) & 1u)) acc[i][j][e] = 0.0f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (mb + e >= g.M || !col_ok) acc[i][j][e] = 0.0f;
        if (EPI == EPI_FWD) {
#pragma unroll
          for (int e = 0; e < 4; ++e) word |= (uint32_t)((float)(bf16)acc[i][j][e] > 0.0f) << (4 * i + e);
          __builtin_amdgcn_sched_barrier(0);     // one block's conversions at a time: hoisted together they cost registers
        }
      }
      // the mask the data gradient of the layer above will need: one bit per stored (bf16-rounded) output > 0
      if (EPI == EPI_FWD && g.bits_out && col_ok && rowW < g.M) g.bits_out[(size_t)n * g.ldbits + (rowW >> 5) + lgrp] = word;
      __builtin_amdgcn_sched_barrier(0);
    }
    auto pack4 = [](float a, float b, float c, float d) {
      const bf16x4 o = {(bf16)a, (bf16)b, (bf16)c, (bf16)d};
      return __builtin_bit_cast(u32x2, o);
    };
    if (g.CT) {   // transposed: staged row = output column n; a piece = 8 consecutive rows m of it
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int r = j * 16 + lrow;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int mloc = i * 16 + 4 * lgrp;     // 8 bytes at element mloc of the staged row
          *(u32x2*)(reg + r * 256 + (((mloc >> 3) ^ (r & 15)) << 4) + (mloc & 4) * 2) =
              pack4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        }
      }
#pragma unroll
      for (int it = 0; it < 16; ++it) {
        const int r = it * 4 + (lane >> 4), c = lane & 15;
        const int n = colW + r, m = rowW + c * 8;
        const u32x4 val = *(const u32x4*)(reg + r * 256 + ((c ^ (r & 15)) << 4));
        if (n < g.N && m < Mr) *(u32x4*)((bf16*)g.CT + (size_t)n * g.ldct + m) = val;
      }
    }
    if (g.C) {    // row-major: after the 4x4 transpose inside lane quads a lane holds 4 consecutive columns of one row
#pragma unroll
      for (int j = 0; j < NB; ++j) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[i][j][e];
          quad_transpose(v, lane);
          const int r = i * 16 + 4 * lgrp + (lane & 3);
          const int nloc = j * 16 + (lrow & ~3);
          *(u32x2*)(reg + r * 128 + (((nloc >> 3) ^ ((r >> 1) & 7)) << 4) + (nloc & 4) * 2) = pack4(v[0], v[1], v[2], v[3]);
        }
      }
#pragma unroll
      for (int it = 0; it < 16; ++it) {
        const int r = it * 8 + (lane >> 3), c = lane & 7;
        const int m = rowW + r, n = colW + c * 8;
        const u32x4 val = *(const u32x4*)(reg + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
        if (m < g.M && n < g.N) *(u32x4*)((bf16*)g.C + (size_t)m * g.ldc + n) = val;
      }
    }
  }
#endif
}

// f(0), f(1), ... f(N - 1) with the index as a constant.
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// The order in which gemm_nt_long_kernel multiplies the 8 A fragments of a sub-step with its 8 B fragments: strips of two A rows, down the
// columns and back up, so that from one MFMA to the next one operand changes, A and B in turn, and each is used again within two.  The chip is
// power-limited here.  Milliseconds with one A fragment against all of B's, back and forth / strips of 4 / of 2: forward 8192 x 16384 x
// 16384 2.793 / 2.787 / 2.763, data gradient 2.784 / 2.782 / 2.760, weight gradient 16384 x 16384 x 8192 2.937 / 2.912 / 2.902; pairs of columns
// instead of rows the same.
struct LongWalk {
  int a[64], b[64], first[16];     // fragments of MFMA m; all fragments (0 .. 7 A, 8 .. 15 B) in the order of their first use
  constexpr LongWalk() : a(), b(), first() {
    for (int m = 0; m < 64; ++m) {
      const int strip = m / 16, c = m % 16 / 2;
      a[m] = 2 * strip + (c & 1 ? 1 - m % 2 : m % 2);
      b[m] = strip & 1 ? 7 - c : c;
    }
    bool seen[16] = {};
    for (int m = 0, n = 0; m < 64; ++m)
      for (int f : {a[m], 8 + b[m]})
        if (!seen[f]) {
          seen[f] = true;
          first[n++] = f;
        }
  }
};

// The same 256x256 tile for long contractions (see big_is_long): 4 wavefronts of 128 x 128, one per SIMD, accumulators in 256 AGPRs.  Per
// k-tile they read 128 KB of fragments from LDS where 8 wavefronts of 128 x 64 read 192, in a third fewer instructions, and what the chip saves
// there it spends on a higher clock.  With one wavefront on a SIMD nothing else fills its issue slots: an MFMA takes the matrix pipe 16 cycles, so
// between two of them there is room for about three other instructions, and any place with more of them is lost time.  So the k-loop has at
// most two: fragment reads at every second or third MFMA, and loads whose LDS address (m0) is set in front of an MFMA and whose offset
// holds nothing but one register and one scalar, every sixth (builtins with their address arithmetic in one place cost 160 cycles a k-tile).
// The MFMAs are written as assembly so that the accumulators stay where they are: the register allocator otherwise moves a quarter of
// them between VGPRs and AGPRs in every k-tile.
// A k-tile is 128 MFMAs, m = 0 .. 63 of k-sub-step 0, then of 1; all 16 fragments of a sub-step are in registers before it starts:
//   MFMA   0 ..  30   reads of sub-step 1
//         40          barrier X: nobody reads this k-tile's stage any more
//         42 .. 132   the 16 loads of k-tile kt + 2 into that stage (the last one in the next k-tile's time)
//         79          barrier Y: k-tile kt + 1 has landed
//         80 .. 125   reads of its sub-step 0
// Cycles per k-tile, 8192 x 16384 x 16384 (2048 of them MFMAs), one A fragment against all of B's at a time: 2170 with no loads, 2260 with loads past the operands, 2310 with loads that all hit
// the L2, 2430-2460 as it is; the kernel above 2360-2390 at a clock 5-8 % lower.
// At the loop's head the compiler waits for every LDS read, and the first one of sub-step 1 has just gone out before that wait: one LDS latency a k-tile
// that nothing on the SIMD covers.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_nt_long_kernel(const GemmArgs g) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef bf16 T;
  typedef __attribute__((ext_vector_type(4))) int i32x4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __builtin_amdgcn_s_setprio(3);
  constexpr int BM = 256, BN = 256, ES = 2, CH = 8, BK = 64;
  constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
  constexpr int RD1 = 0, X = 40, LD = 42, LD_STEP = 6, Y = 79, RD0 = 80;      // MFMA index of what the comment above lists
  constexpr int kOwn = (128 - LD + LD_STEP - 1) / LD_STEP;                    // loads of a k-tile that do not go out in the next one's time
  constexpr int kBeforeY = (Y - LD + LD_STEP - 1) / LD_STEP;                  // loads of k-tile kt + 2 that are out at barrier Y
  static_assert(kOwn <= 16 && LD > X && LD + 15 * LD_STEP - 128 < X && RD1 + 2 * 15 < X && RD0 + 3 * 15 < 128, "order of the events of a k-tile");
  int tm, tn;
  big_tile(g, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wm = w & 1, wn = w >> 1;
  const int lgrp = lane >> 4, lrow = lane & 15;

  const int Kr = (g.K + CH - 1) / CH * CH;
  const int nk = (Kr + BK - 1) / BK;
  // the buffer resource by words: as an operand of assembly it has to be a vector
  auto rsrc_of = [](const void* p, size_t bytes) {
    const uint64_t a = (uint64_t)(uintptr_t)p;
    return i32x4{(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)bytes, 0x00020000};
  };
  const i32x4 rsrcA = rsrc_of(g.A, (size_t)g.M * g.lda * ES), rsrcB = rsrc_of(g.B, (size_t)g.N * g.ldb * ES);
  // load i < 8 fills rows [32 i, 32 i + 32) of A's tile, i >= 8 of B's; wavefront w rows 8w .. 8w + 7 of those
  const int prow = w * 8 + (lane >> 3);
  const int pchunk = (lane & 7) ^ ((prow >> 1) & 7);
  uint32_t voff[16];
#pragma unroll
  for (int i = 0; i < 8; ++i) voff[i] = (uint32_t)(((size_t)(m0 + prow + 32 * i) * g.lda + pchunk * CH) * ES);
#pragma unroll
  for (int i = 0; i < 8; ++i) voff[8 + i] = (uint32_t)(((size_t)(n0 + prow + 32 * i) * g.ldb + pchunk * CH) * ES);
  typedef __attribute__((address_space(3))) void* lds_ptr_t;
  const uint32_t lds_wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(uintptr_t)(lds_ptr_t)smem + w * 8 * 128));

  // what the epilogue reads, ahead of the operands
  const int rowW = m0 + wm * 128, colW = n0 + wn * 128;
  float bias[8];
  uint32_t mbits[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int n = colW + j * 16 + lrow;
    bias[j] = 0.0f;
    mbits[j] = EPI == EPI_DGRAD && !g.bits ? 0xFFFFFFFFu : 0u;
    if (EPI == EPI_FWD && n < g.N) bias[j] = g.bias[n];
    if (EPI == EPI_DGRAD && g.bits && n < g.N && rowW < g.M) mbits[j] = g.bits[(size_t)n * g.ldbits + (rowW >> 5) + lgrp];
  }

  f32x4 acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

  // Chunks past K become zero fills: one that is past it in a k-tile is past it in all that follow.
  auto clip = [&](int kt) {
    if (kt * BK + BK > Kr) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (kt * BK + pchunk * CH >= Kr) voff[i] = kOutOfRange;
    }
  };
  // The k offset is a scalar; k-tiles past the end, whose offsets are out of range already, take 0, so that no sum of the two wraps.
  auto koff_of = [&](int kt) { return (uint32_t)(kt < nk ? kt : 0) * 128u; };
  // The statements name the m0 they set, so that one set by the compiler for an access of its own does not pass for still set behind them; it
  // warns of every register it reserves.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
#define SLP_LOAD "s_add_u32 m0, %[base], %[row]\n\t"
#define SLP_LOAD_ARGS(i, base_, koff_)                                                                                             \
  [base] "s"(base_), [row] "i"((i) < 8 ? (i) * 4096 : A_BYTES + ((i) - 8) * 4096), [off] "v"(voff[i]), [rsrc] "s"((i) < 8 ? rsrcA : rsrcB), \
      [koff] "s"(koff_)
  auto load = [&](int i, uint32_t base, uint32_t koff) {
    asm volatile(SLP_LOAD "s_nop 1\n\tbuffer_load_dwordx4 %[off], %[rsrc], %[koff] offen lds" : : SLP_LOAD_ARGS(i, base, koff) : "memory", "scc", "m0");
  };
  u32x4 af[2][8], bfr[2][8];
  uint32_t fa[2], fb[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const uint32_t xo = (uint32_t)(((kk * 4 + lgrp) ^ ((lane >> 1) & 7)) << 4);
    fa[kk] = (uint32_t)((wm * 128 + lrow) * 128) + xo;
    fb[kk] = (uint32_t)(A_BYTES + (wn * 128 + lrow) * 128) + xo;
  }
  constexpr LongWalk walk;
  auto read = [&](int stage, int kk, int f) {
    if (f < 8) af[kk][f] = *(const u32x4*)(smem + stage * STAGE + fa[kk] + f * 2048);
    else bfr[kk][f - 8] = *(const u32x4*)(smem + stage * STAGE + fb[kk] + (f - 8) * 2048);
  };
  auto mma = [&](int kk, int ia, int ib) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[ia][ib]) : "v"(af[kk][ia]), "v"(bfr[kk][ib]));
  };
  auto mma_load = [&](int kk, int ia, int ib, int i, uint32_t base, uint32_t koff) {        // the MFMA is the wait state that m0 needs
    asm volatile(SLP_LOAD "v_mfma_f32_16x16x32_bf16 %[acc], %[a], %[b], %[acc]\n\tbuffer_load_dwordx4 %[off], %[rsrc], %[koff] offen lds"
                 : [acc] "+a"(acc[ia][ib]) : [a] "v"(af[kk][ia]), [b] "v"(bfr[kk][ib]), SLP_LOAD_ARGS(i, base, koff) : "memory", "scc", "m0");
  };
#define SLP_FENCE() __builtin_amdgcn_sched_barrier(0)
#define SLP_BARRIER(cnt)                                            \
  do {                                                              \
    __builtin_amdgcn_s_waitcnt(cnt);                                \
    asm volatile("" ::: "memory");                                  \
    __builtin_amdgcn_s_barrier();                                   \
    asm volatile("" ::: "memory");                                  \
  } while (0)
  constexpr int kLgkm0 = 0xC07F;         // every LDS read has returned
  clip(0);
  static_for<16>([&](auto i) { load(i, lds_wave, 0u); });
  clip(1);
  static_for<kOwn>([&](auto i) { load(i, lds_wave + STAGE, koff_of(1)); });
  SLP_BARRIER(SLP_VMCNT(kOwn));
#pragma unroll
  for (int f = 0; f < 16; ++f) read(0, 0, f);
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1, nxt = cur ^ 1;
    const uint32_t base1 = lds_wave + nxt * STAGE, base2 = lds_wave + cur * STAGE, koff1 = koff_of(kt + 1), koff2 = koff_of(kt + 2);
    static_for<128>([&](auto pc) {
      constexpr int p = decltype(pc)::value, kk = p / 64, ia = walk.a[p % 64], ib = walk.b[p % 64], late = p + 128 - LD, own = p - LD;
      if constexpr (p == X) {
        SLP_BARRIER(kLgkm0);
        clip(kt + 2);
      }
      if constexpr (p == Y) SLP_BARRIER(SLP_VMCNT(kBeforeY));
      if constexpr (p >= RD1 && (p - RD1) % 2 == 0 && (p - RD1) / 2 < 16) read(cur, 1, walk.first[(p - RD1) / 2]);
      if constexpr (p >= RD0 && (p - RD0) % 3 == 0 && (p - RD0) / 3 < 16) read(nxt, 0, walk.first[(p - RD0) / 3]);
      if constexpr (late % LD_STEP == 0 && late / LD_STEP < 16) mma_load(kk, ia, ib, late / LD_STEP, base1, koff1);
      else if constexpr (own >= 0 && own % LD_STEP == 0 && own / LD_STEP < 16) mma_load(kk, ia, ib, own / LD_STEP, base2, koff2);
      else mma(kk, ia, ib);
      SLP_FENCE();
    });
  }
  // the last zero fills have landed, and the matrix pipe is done with the accumulators (the compiler does not see MFMAs in assembly)
  __builtin_amdgcn_s_waitcnt(SLP_VMCNT(0));
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
  for (int i = 0; i < 64; ++i) asm volatile("" : "+a"(acc[i / 8][i % 8]));
#undef SLP_FENCE
#undef SLP_BARRIER
#undef SLP_LOAD
#undef SLP_LOAD_ARGS
#pragma clang diagnostic pop

  if constexpr (EPI == EPI_WGRAD) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int n = n0 + wn * 128 + j * 16 + lrow;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float v[4];
        asm volatile("" : "+a"(acc[i][j]));        // one block at a time leaves the AGPRs
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][e];
        store_quad<T, EPI>(g, n, m0 + wm * 128 + i * 16 + 4 * lgrp, 0.0f, v, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    // Forward / data gradient: a wavefront stages its 128 x 128 sub-tile in a private 32 KB of the stages, transposed (128 rows n of 256
    // bytes), and takes both layouts out of it: whole rows, and, through transposing LDS reads (a group of 16 lanes reads 4 rows of 16
    // columns, lane l gets the 4 values of column l), pieces of 16 bytes of 64-byte row segments of the row-major output.  16-byte chunk c of
    // staged row n sits at c ^ swz(n): 16 rows in a row lie on 16 chunks, and the 8 rows that half a wavefront reads transposed, 0 .. 3 and 8 .. 11
    // or 4 .. 7 and 12 .. 15, on disjoint ones.  A row-major copy staged on its own took 16 more instructions a block for the transpose
    // inside lane quads and half of the staging's LDS writes.
    typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
    typedef __attribute__((ext_vector_type(4))) short i16x4;
    typedef __attribute__((address_space(3))) i16x4* lds_i16x4;
    const bool edge = rowW + 128 > g.M || colW + 128 > g.N;      // uniform over the wavefront
    const int Mr = (g.M + 7) & ~7;
    __syncthreads();
    unsigned char* const st = smem + w * 32768;
    auto swz = [](int n) { return ((n & 3) << 1) | (n & 8) | ((n >> 2) & 1); };
    unsigned char* const wbase = st + lrow * 256 + (lgrp & 1) * 8;
    const int wsw = (lgrp >> 1) ^ swz(lrow);
    const bool relu = EPI == EPI_FWD && g.relu;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int n = colW + j * 16 + lrow;
      const bool col_ok = n < g.N;
      uint32_t xw[2] = {0, 0};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int mb = rowW + i * 16 + 4 * lgrp;
        float v[4];
        asm volatile("" : "+a"(acc[i][j]));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][e];
        if (EPI == EPI_FWD) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += bias[j];
          if (relu) {
#pragma unroll
            for (int e = 0; e < 4; ++e) asm("v_max_f32 %0, 0, %1" : "=v"(v[e]) : "v"(v[e]));
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            v[e] = __builtin_bit_cast(float, __builtin_bit_cast(int, v[e]) & (((int)(mbits[j] << (31 - 4 * i - e))) >> 31));
        }
        if (edge) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (mb + e >= g.M || !col_ok) v[e] = 0.0f;
        }
        const bf16x4 o = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
        const u32x2 pk = __builtin_bit_cast(u32x2, o);
        *(u32x2*)(wbase + j * 4096 + ((wsw ^ (2 * i)) << 4)) = pk;
        if (EPI == EPI_FWD) {
          uint32_t lo, hi;                         // 1 in each half that holds a positive value
          asm("v_pk_max_i16 %0, %1, 0\n\tv_pk_min_i16 %0, %0, %2" : "=&v"(lo) : "v"(pk[0]), "s"(0x00010001));
          asm("v_pk_max_i16 %0, %1, 0\n\tv_pk_min_i16 %0, %0, %2" : "=&v"(hi) : "v"(pk[1]), "s"(0x00010001));
          xw[i >> 2] |= (lo | (hi << 2)) << (4 * (i & 3));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (EPI == EPI_FWD && g.bits_out && col_ok && rowW < g.M) {
        uint32_t word = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) word |= ((xw[q] & 0x5555u) | ((xw[q] >> 15) & 0xAAAAu)) << (16 * q);
        g.bits_out[(size_t)n * g.ldbits + (rowW >> 5) + lgrp] = word;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // 8 pieces at a time: their LDS reads are under way together
    if (g.CT) {
      const int r0 = lane >> 4, c = lane & 15, m = rowW + c * 8;
      bf16* const out = (bf16*)g.CT + (size_t)(colW + r0) * g.ldct + m;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        u32x4 val[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int r = (8 * b + q) * 4 + r0;
          val[q] = *(const u32x4*)(st + r * 256 + ((c ^ swz(r & 15)) << 4));
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int r = (8 * b + q) * 4;
          if (!edge || (colW + r + r0 < g.N && m < Mr)) *(u32x4*)(out + (size_t)r * g.ldct) = val[q];
        }
      }
    }
    if (g.C) {
      const int gq = lane >> 4, jj = lane & 15;
      const int r0 = gq * 8 + (jj >> 2);                           // staged row of the first of the two reads
      const uint32_t base = (uint32_t)(r0 * 256 + ((((jj & 3) >> 1) ^ swz(r0 & 15)) << 4) + (jj & 1) * 8);
      const int n = colW + gq * 8;
      bf16* const out = (bf16*)g.C + (size_t)(rowW + jj) * g.ldc + n;
#pragma unroll
      for (int b = 0; b < 8; b += 2) {
        u32x2 val[8][2];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const uint32_t o1 = (base ^ ((b + q / 4) << 5)) + q % 4 * 8192;
          val[q][0] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4)(st + o1)));
          val[q][1] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4)(st + ((o1 ^ 16) + 1024))));
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int r = (b + q / 4) * 16, c = q % 4 * 32;
          if (!edge || (rowW + jj + r < g.M && n + c < g.N))
            *(u32x4*)(out + (size_t)r * g.ldc + c) = u32x4{val[q][0][0], val[q][0][1], val[q][1][0], val[q][1][1]};
        }
      }
    }
  }
#endif
}

// ---- host side -------------------------------------------------------------------------------
struct TileCfg { int bm, bn; const char* name; };
const TileCfg kCfgs[3] = {{256, 256, "256x256"}, {128, 128, "128x128"}, {64, 64, "64x64"}};
constexpr int kCfg128TwoStage = 3, kCfg128x64 = 4;

long tiles_of(int M, int N, int c) {
  return (long)((M + kCfgs[c].bm - 1) / kCfgs[c].bm) * ((N + kCfgs[c].bn - 1) / kCfgs[c].bn);
}

// The tile configuration of a product: the largest tile that still gives most of the 256 compute units work.
int pick_cfg(int dtype, int epi, int M, int N) {
  const long t128 = tiles_of(M, N, 1);
  if (tiles_of(M, N, 0) >= 224) return 0;
  // 128x128 with two 32 KB stages lets two workgroups share a compute unit, four stages of one workgroup are faster as long as
  // every tile has a unit of its own.  bf16, microseconds with four / two stages: 1024x4096x4096 (256 tiles) 32 / 48,
  // 3001x1500x1000 (288) 21.6 / 19.2, 1500x3500x1000 (336) 25.7 / 23.4, 2500x2500x1000 (400) 26.3 / 23.1, 2048x4096x1024
  // (512) 23.4 / 19.4.  float32, bound by the matrix pipe: 2048x2048x1024 (256) 71 / 73.
  const int cfg128 = t128 > (dtype == 1 ? 256 : 511) ? kCfg128TwoStage : 1;
  if (dtype == 1 && (epi == EPI_FWD || epi == EPI_DGRAD)) {
    // More than half of the units busy with 128x128 tiles beat all of them on 64x64 ones, whose operands take twice the way
    // into LDS per product: 1280x1664x1024 (130 tiles) 13.7 against 15.4 us, 1000x3001x1500 (192) 17.1 against 20.4.  Below
    // that 128x64 tiles, if they come to most of 256: 1000x1500x3001 (192) 19.6 against 21.6 on 64x64, 1024x2048x4096 (256)
    // 24.0 against 29.2; 1000x777x3001 (104) 18.3 against 14.3.
    if (t128 > 128) return cfg128;
    const long t = (long)((M + 127) / 128) * ((N + 63) / 64);
    return t >= 176 && t <= 256 ? kCfg128x64 : 2;
  }
  // weight gradients (the kernel for small layers takes the update along) and float32
  return t128 >= 224 ? cfg128 : 2;
}

template <typename T, int BM, int BN, int EPI, int NW, int NS>
hipError_t configure_one() {
  constexpr int smem = NS * (BM + BN) * 128;
  static std::once_flag once;       // one attribute call per instantiation, also when two host threads launch first together
  static hipError_t result = hipSuccess;
  std::call_once(once, [] {
    result = hipFuncSetAttribute((const void*)gemm_nt_kernel<T, BM, BN, EPI, NW, NS>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  return result;
}

template <typename T, int BM, int BN, int EPI, int NW, int NS>
hipError_t launch_one(const GemmArgs& g, hipStream_t s) {
  constexpr int smem = NS * (BM + BN) * 128;
  auto kern = gemm_nt_kernel<T, BM, BN, EPI, NW, NS>;
  hipError_t e = configure_one<T, BM, BN, EPI, NW, NS>();
  if (e != hipSuccess) return e;
  const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(NW * 64), smem, s, g);
  return hipGetLastError();
}

constexpr int kBigWaves = 8;
constexpr int kBigSmem = 2 * 512 * 128;

template <int EPI>
hipError_t configure_big() {
  static std::once_flag once;
  static hipError_t result = hipSuccess;
  std::call_once(once, [] {
    result = hipFuncSetAttribute((const void*)gemm_nt_big_kernel<EPI, kBigWaves>, hipFuncAttributeMaxDynamicSharedMemorySize, kBigSmem);
  });
  return result;
}

// Whether the 256x256 tiles of a product run on 4 wavefronts (gemm_nt_long_kernel) instead of 8: from a length of the contraction on from which
// the cheaper k-tiles outweigh an epilogue in which one wavefront a SIMD waits for its own LDS reads.  What they save is power: on a chip that the last
// round of tiles leaves mostly empty the clock is not the limit and the 8 wavefronts are faster for longer.  Microseconds, 8 / 4 wavefronts:
//   full rounds: forward 8192 x 8192, K = 1024 146 / 149, 2048 225 / 221, 8192 x 16384, 2048 461 / 449, 16384 2890 / 2770, 7680 x 8192 (960 tiles),
//   3072 288 / 275; data gradient 8192 x 16384, 2048 455 / 456, 7680 x 8192, 3072 288 / 275, 4096 x 12000 (752), 3072 214 / 208; weight gradient 8192 x
//   8192, 3072 321 / 314, 16384 x 16384 x 8192 3075 / 2945;
//   others: forward 4352 x 4352 (289), 3072 128 / 130, 4096 163 / 163, 6144 231 / 229, 12000 x 4100 (799), 3072 261 / 263, 4096 334 / 332; data gradient
//   4352 x 4352, 3072 126 / 129, 4096 160 / 162, 6144 229 / 229, 8192 298 / 295, 12000 x 4100, 3072 257 / 265, 4096 332 / 335, 6144 480 / 472; weight
//   gradient 4352 x 4352, 3072 126 / 125, 4096 160 / 158.
bool big_is_long(int epi, int M, int N, int K) {
  const long tiles = tiles_of(M, N, 0), rounds = (tiles + 255) / 256;
  if (epi == EPI_WGRAD || 8 * tiles >= 7 * 256 * rounds) return K >= 3072;
  return K >= (epi == EPI_FWD ? 4096 : 6144);
}

template <int EPI>
hipError_t configure_long() {
  static std::once_flag once;
  static hipError_t result = hipSuccess;
  std::call_once(once, [] {
    result = hipFuncSetAttribute((const void*)gemm_nt_long_kernel<EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, kBigSmem);
  });
  return result;
}

template <int EPI>
hipError_t launch_big(const GemmArgs& g, hipStream_t s) {
  constexpr int smem = kBigSmem;
  const int tiles = ((g.M + 255) / 256) * ((g.N + 255) / 256);
  if constexpr (EPI != EPI_WGRAD_UPDATE) {
    if (big_is_long(EPI, g.M, g.N, g.K)) {
      hipError_t e = configure_long<EPI>();
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(gemm_nt_long_kernel<EPI>, dim3(tiles), dim3(256), smem, s, g);
      return hipGetLastError();
    }
  }
  hipError_t e = configure_big<EPI>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((gemm_nt_big_kernel<EPI, kBigWaves>), dim3(tiles), dim3(kBigWaves * 64), smem, s, g);
  return hipGetLastError();
}

// LDS stages of gemm_nt_kernel (loads run stages-1 k-tiles ahead of the multiplies): a 256x256 tile fills LDS with two;
// the k-tiles of the small tiles are 4-16x shorter, too short to cover the loads of the next one, so they keep four.
template <typename T, int EPI>
hipError_t launch_cfg(int cfg, const GemmArgs& g, hipStream_t s) {
  switch (cfg) {
    case 0:
      if constexpr (sizeof(T) == 2) return launch_big<EPI>(g, s);
      else return launch_one<T, 256, 256, EPI, 8, 2>(g, s);
    case 1: return launch_one<T, 128, 128, EPI, 8, 4>(g, s);     // 8 wavefronts of 64x32: +5-10 % over 4 of 64x64 here
    case kCfg128TwoStage: return launch_one<T, 128, 128, EPI, 4, 2>(g, s);
    case kCfg128x64:
      if constexpr (sizeof(T) == 2 && (EPI == EPI_FWD || EPI == EPI_DGRAD)) return launch_one<T, 128, 64, EPI, 8, 4>(g, s);
      else return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;     // (small products are launched before the switch)
  }
}

template <typename T>
hipError_t launch_epi(int epi, int cfg, const GemmArgs& g, hipStream_t s) {
  switch (epi) {
    case EPI_FWD: return launch_cfg<T, EPI_FWD>(cfg, g, s);
    case EPI_DGRAD: return launch_cfg<T, EPI_DGRAD>(cfg, g, s);
    case EPI_WGRAD_UPDATE: return launch_cfg<T, EPI_WGRAD_UPDATE>(cfg, g, s);
    default: return launch_cfg<T, EPI_WGRAD>(cfg, g, s);
  }
}

template <typename T, int EPI>
hipError_t configure_epi() {
  hipError_t e;
  if constexpr (sizeof(T) == 2) {
    e = configure_big<EPI>();
    if constexpr (EPI != EPI_WGRAD_UPDATE)
      if (e == hipSuccess) e = configure_long<EPI>();
  } else e = configure_one<T, 256, 256, EPI, 8, 2>();
  if (e == hipSuccess) e = configure_one<T, 128, 128, EPI, 8, 4>();
  if (e == hipSuccess) e = configure_one<T, 128, 128, EPI, 4, 2>();
  if constexpr (sizeof(T) == 2 && (EPI == EPI_FWD || EPI == EPI_DGRAD)) {
    if (e == hipSuccess) e = configure_one<T, 128, 64, EPI, 8, 4>();
  }
  return e;
}

}  // namespace

// One-time kernel attributes of every instantiation, so that no launch has to set one later
// (a launch sequence that is being captured into a graph should consist of launches only).
hipError_t gemm_configure_all() {
  hipError_t e = configure_epi<bf16, EPI_FWD>();
  if (e == hipSuccess) e = configure_epi<bf16, EPI_DGRAD>();
  if (e == hipSuccess) e = configure_epi<bf16, EPI_WGRAD>();
  if (e == hipSuccess) e = configure_epi<bf16, EPI_WGRAD_UPDATE>();
  if (e == hipSuccess) e = configure_epi<float, EPI_FWD>();
  if (e == hipSuccess) e = configure_epi<float, EPI_DGRAD>();
  if (e == hipSuccess) e = configure_epi<float, EPI_WGRAD>();
  if (e == hipSuccess) e = configure_epi<float, EPI_WGRAD_UPDATE>();
  if (e == hipSuccess) e = small_configure_all();
  if (e == hipSuccess) e = pair_configure_all();
  if (e == hipSuccess) e = chain_configure_all();
  return e;
}

// Whether launch_pair may take the product: the sums of its 128x128 tiles are in the order of every tile but the 16 and 32 ones, whose
// products are better off in a group of their kind; 256x256 tiles are faster where there are enough of them.
bool product_can_pair(int dtype, int epi, int M, int N) {
  const int c = pick_cfg(dtype, epi, M, N);
  return c != 0 && !(c == 2 && small_tile(dtype, M, N) < 64);
}

// Whether the 256x256 tiles of an output are whole rounds of the 256 compute units.
bool product_fills_rounds(int M, int N) { return tiles_of(M, N, 0) % 256 == 0; }

bool product_is_small(int dtype, int epi, int M, int N) { return pick_cfg(dtype, epi, M, N) == 2; }

const char* gemm_config_name(int dtype, int M, int N, int K) {
  (void)K;
  const int c = pick_cfg(dtype, EPI_FWD, M, N), t = small_tile(dtype, M, N);
  if (c == 2 && t < 64) return t == 16 ? "16x16 k-split" : "32x32 k-split";
  if (c == kCfg128x64) return "128x64";
  return c == kCfg128TwoStage ? "128x128 (2 stages)" : kCfgs[c].name;
}

hipError_t launch_gemm(int dtype, int epi, const GemmArgs& g, hipStream_t s) {
  const int es = dtype == 1 ? 2 : 4;
  // the kernel addresses operands with 32-bit byte offsets and a 2 GiB sentinel
  if ((size_t)g.M * g.lda * es >= 0x80000000ull || (size_t)g.N * g.ldb * es >= 0x80000000ull) return hipErrorInvalidValue;
  if (g.lda % kLdAlign || g.ldb % kLdAlign || g.M <= 0 || g.N <= 0 || g.K <= 0) return hipErrorInvalidValue;
  if (!g.A || !g.B) return hipErrorInvalidValue;                      // a missing operand must never reach the device
  if (((uintptr_t)g.A | (uintptr_t)g.B) & 15) return hipErrorInvalidValue;
  if (epi == EPI_FWD && !g.bias) return hipErrorInvalidValue;
  if (epi == EPI_WGRAD && !g.Cf) return hipErrorInvalidValue;
  if (epi == EPI_WGRAD_UPDATE) {
    if (!g.uW || !g.uV || g.ldc % 4 || (((uintptr_t)g.uW | (uintptr_t)g.uV | (uintptr_t)g.uW16 | (uintptr_t)g.uWT) & 15)) return hipErrorInvalidValue;
    if (g.uWT && g.ldwt % kLdAlign) return hipErrorInvalidValue;
  }
  if (epi != EPI_WGRAD && epi != EPI_WGRAD_UPDATE && !g.C && !g.CT) return hipErrorInvalidValue;
  // outputs are written as 16-byte vectors
  if (epi != EPI_WGRAD && epi != EPI_WGRAD_UPDATE && ((g.C && (g.ldc % kLdAlign || ((uintptr_t)g.C & 15))) || (g.CT && (g.ldct % kLdAlign || ((uintptr_t)g.CT & 15)))))
    return hipErrorInvalidValue;
  if (epi == EPI_WGRAD && (g.ldc % 4 || ((uintptr_t)g.Cf & 15))) return hipErrorInvalidValue;
  const int cfg = pick_cfg(dtype, epi, g.M, g.N);
  if (cfg == 0 && dtype == 1 && epi == EPI_DGRAD && g.maskT && !g.bits) return hipErrorInvalidValue;      // 256x256 bf16 tiles read the mask as bits only
  if (cfg == 2) {
    SmallGroup one{};
    one.g[0] = g; one.epi[0] = epi; one.n = 1;
    return launch_small_group(dtype, one, s);
  }
  GemmArgs h = g;
  // Height of the tile groups each XCD walks (the 32 tiles an XCD runs together are group_m tile rows x 32/group_m
  // tile columns).  8 is best everywhere except the weight gradient of a tall output (64 or more tile rows), whose
  // float32 rows are written faster when the concurrent tiles are wider than tall: measured 3.61 -> 3.47 ms on
  // 16384x16384x8192 and 1.90 -> 1.82 ms on 16384x8192x8192, no gain or a loss on every other shape tried.
  h.group_m = ((epi == EPI_WGRAD || epi == EPI_WGRAD_UPDATE) && cfg == 0 && (g.M + 255) / 256 >= 64) ? 4 : kGroupM;
  // Big bf16 products whose tile grid divides into 16 x 16 regions take the region walk instead: equal or better than
  // either group height on every shape tried (+1-4 %; +14 % on the short contraction of a first layer, K = 784).
  if (cfg == 0 && dtype == 1 && ((g.M + 255) / 256) % 16 == 0 && ((g.N + 255) / 256) % 16 == 0) h.group_m = kRegionWalk;
  return dtype == 1 ? launch_epi<bf16>(epi, cfg, h, s) : launch_epi<float>(epi, cfg, h, s);
}

}  // namespace slp
