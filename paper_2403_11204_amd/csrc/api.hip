// C ABI of the segment-training library (see include/slp.h for the contract).
// Host code only: argument validation, the device-memory carve-up of the two
// caller-provided buffers, and the launch sequence of one training step
// (paper Sec. 2: a segment is trained on its own inputs and targets, nothing
// flows to or from another segment).
#include "../../include/slp.h"

#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "slp_kernels.h"

using namespace slp;

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

#define HIP_TRY(expr)                                                                             \
  do {                                                                                            \
    hipError_t e__ = (expr);                                                                      \
    if (e__ != hipSuccess) return fail(SLP_ERR_DEVICE, "%s: %s", #expr, hipGetErrorString(e__)); \
  } while (0)

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Layer {
  int K, N;        // fan-in, fan-out
  int ldk, ldn;    // padded leading dimensions of [N][ldk] and [K][ldn] matrices
  // offsets into the parameter buffer
  size_t oW32, ovW, odW, ob, ovb, odb, oW16, oWT;
  // bound pointers
  float *W32, *vW, *dW, *b, *vb, *db;
  void *Wop;       // forward operand: W16 (bf16 mode) or W32
  void *W16;       // bf16 copy or null
  void *WT;        // [K][ldn] transposed copy for the data gradient, null for the first layer
};

struct ProfRec { hipEvent_t a, b; double flops; };

// One captured training step: the launch sequence depends on these arguments only
// (every other kernel argument is fixed once the handle is bound).
struct StepGraph {
  const void* X;
  const int32_t* targets;
  int batch;
  float* loss_out;
  hipGraphExec_t exec;
  uint64_t used;
};
constexpr size_t kMaxStepGraphs = 16;
// Steps of at most this many launches are launched one by one even where graphs are on: starting a graph costs the host more
// than that many launches, and the device as much between its kernels.  Replayed / one by one, microseconds a step: 784-128-64
// batch 64 (4 launches) 25.8 / 18.5, 784-80-60 batch 1410 (4) 31.7 / 26.7, 512-1024-1024-47 batch 256 (7) 65 / 60; layers of 64,
// batch 64, 5 launches 26.8 / 19.0, 6 28.0 / 21.6, 7 30.5 / 24.0, 8 31.4 / 26.7, 9 35.0 / 30.6, 10 37.2 / 33.1, 13 47.0 / 43.4.
// One by one keeps its 4 us beyond the line on an idle host; on a busy one (the same in another run) 11 launches took 41.1 /
// 52.5 and 12 43.1 / 55.8, and up to 10 nothing, so the line leaves the host some room.
constexpr int kDirectLaunches = 8;

}  // namespace

struct slp_segment {
  int L, act, loss, dtype, max_batch, ldb;   // ldb: leading dimension of batch-contiguous buffers
  float lr, mu;
  std::vector<int> widths, ldw;              // ldw[l] = padded width l
  std::vector<Layer> layers;
  size_t param_bytes, work_bytes;
  // workspace offsets / pointers, index = layer 0..L
  std::vector<size_t> oA, oAT, odZ, odZT, oBits;
  std::vector<void*> A, AT, dZ, dZT;
  std::vector<uint32_t*> bits;   // bf16 mode: [A_l > 0] of the hidden activations, one bit per element (GemmArgs::bits)
  int ldbits;
  size_t oPartials, oLoss, oBadIds, oHurry;
  int n_partials;
  float *partials, *loss_dev;
  unsigned* hurry;                           // device flag that ends the pauses of paced updates (see settle)
  bool paced;                                // updates pending that are paced and have not been told to hurry
  unsigned* bad_ids;                         // rows whose class id was out of range, counted by the loss kernels
  bool bound, have_params;
  bool input_grad;                           // keeps W_1^T and a dZ_0 buffer so that d loss / d input can be formed
  const float* table;
  int classes;
  int last_batch;
  bool prof;
  std::vector<ProfRec> prof_log;
  std::vector<hipEvent_t> ev_pool;
  // The parameter update of layer l is memory-bound and independent of the matrix products of the
  // layers below it, so where it is not part of its own product's launch (see update_in_product) it runs on a side stream next to
  // them (fork after the weight gradient of layer l, join at the end of the step: the caller's stream still orders
  // everything).
  hipStream_t side;
  std::vector<hipEvent_t> ev_fork;   // one per layer
  hipEvent_t ev_join;
  // slp_segment_set_overlap: every layer's update goes to the side stream and slp_segment_step leaves the join to the
  // handle's next call that takes a stream (settle), so that the optimiser tail of one segment runs beside whatever
  // the caller enqueues next -- typically the step of another segment.
  bool defer_join, join_pending;
  // Whether the pending updates came in the order of the layers, an event behind each (ev_update): the next step waits layer by layer.
  bool pending_by_layer;
  int pending_batch;                         // rows of the step they belong to
  std::vector<hipEvent_t> ev_update;
  // slp_segment_set_fused_update: the weight-gradient product applies the optimiser step in its epilogue; the weight
  // gradient itself is never stored.
  bool fused_update;
  long fused_max_params;                     // layers with more weights than this keep the separate update
  // Small segments are bound by launch latency, not by the GPU: with graphs on, the launch sequence of a step
  // is captured once per (X, targets, batch, loss_out) and replayed as one graph launch afterwards.
  bool use_graph, graph_warm;
  int graph_misses;                          // consecutive steps that found no captured graph
  std::vector<StepGraph> graphs;
  uint64_t graph_tick;
  int64_t graph_steps;                       // steps taken by starting a graph
};

namespace {

int esize(const slp_segment* s) { return s->dtype == SLP_BF16 ? 2 : 4; }

// captured steps hold lr, momentum, the label table and the buffer addresses by value
void drop_graphs(slp_segment* s) {
  if (!s->graphs.empty()) (void)hipDeviceSynchronize();   // a replay may still be running; rare (set-up calls only)
  for (auto& g : s->graphs) (void)hipGraphExecDestroy(g.exec);
  s->graphs.clear();
}
bool relu_on(const slp_segment* s, int l) { return l < s->L || s->act == SLP_RELU_ALL; }

hipEvent_t get_event(slp_segment* s) {
  if (!s->ev_pool.empty()) {
    hipEvent_t e = s->ev_pool.back();
    s->ev_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

int run_gemm(slp_segment* s, int epi, const GemmArgs& g, hipStream_t st) {
  ProfRec rec{nullptr, nullptr, 2.0 * g.M * (double)g.N * g.K};
  if (s->prof) {
    rec.a = get_event(s);
    rec.b = get_event(s);
    if (!rec.a || !rec.b) return fail(SLP_ERR_DEVICE, "hipEventCreate failed");
    HIP_TRY(hipEventRecord(rec.a, st));
  }
  HIP_TRY(launch_gemm(s->dtype, epi, g, st));
  if (s->prof) {
    HIP_TRY(hipEventRecord(rec.b, st));
    s->prof_log.push_back(rec);
  }
  return SLP_OK;
}

// The same for a launch of small layers; the time of what rides along in it counts as the products'.
int run_group(slp_segment* s, const SmallGroup& gr, hipStream_t st, bool small = true) {
  ProfRec rec{nullptr, nullptr, 0.0};
  for (int p = 0; p < gr.n; ++p) rec.flops += 2.0 * gr.g[p].M * (double)gr.g[p].N * gr.g[p].K;
  if (s->prof) {
    rec.a = get_event(s);
    rec.b = get_event(s);
    if (!rec.a || !rec.b) return fail(SLP_ERR_DEVICE, "hipEventCreate failed");
    HIP_TRY(hipEventRecord(rec.a, st));
  }
  HIP_TRY(small ? launch_small_group(s->dtype, gr, st) : launch_pair(s->dtype, gr, st));
  if (s->prof) {
    HIP_TRY(hipEventRecord(rec.b, st));
    s->prof_log.push_back(rec);
  }
  return SLP_OK;
}

// The same for a last layer with its cross-entropy.
int run_logits(slp_segment* s, const GemmArgs& g, const OutJob& out, hipStream_t st) {
  ProfRec rec{nullptr, nullptr, 2.0 * g.M * (double)g.N * g.K};
  if (s->prof) {
    rec.a = get_event(s);
    rec.b = get_event(s);
    if (!rec.a || !rec.b) return fail(SLP_ERR_DEVICE, "hipEventCreate failed");
    HIP_TRY(hipEventRecord(rec.a, st));
  }
  HIP_TRY(launch_logits(s->dtype, g, out, st));
  if (s->prof) {
    HIP_TRY(hipEventRecord(rec.b, st));
    s->prof_log.push_back(rec);
  }
  return SLP_OK;
}

// The same for a chain of narrow layers.
int run_chain(slp_segment* s, const ChainLaunch& c, hipStream_t st) {
  ProfRec rec{nullptr, nullptr, 0.0};
  for (int l = 0; l < c.layers; ++l) rec.flops += 2.0 * c.M * (double)c.layer[l].N * (l ? c.layer[l - 1].N : c.K0);
  if (s->prof) {
    rec.a = get_event(s);
    rec.b = get_event(s);
    if (!rec.a || !rec.b) return fail(SLP_ERR_DEVICE, "hipEventCreate failed");
    HIP_TRY(hipEventRecord(rec.a, st));
  }
  HIP_TRY(launch_chain(s->dtype, c, st));
  if (s->prof) {
    HIP_TRY(hipEventRecord(rec.b, st));
    s->prof_log.push_back(rec);
  }
  return SLP_OK;
}

int check_seg(const slp_segment* s, bool need_bound, bool need_params) {
  if (!s) return fail(SLP_ERR_ARG, "segment handle is NULL");
  if (need_bound && !s->bound) return fail(SLP_ERR_STATE, "segment has no device buffers: call slp_segment_bind first");
  if (need_params && !s->have_params)
    return fail(SLP_ERR_STATE, "segment has no parameters: call slp_segment_init or slp_segment_set_params first");
  return SLP_OK;
}

// X[batch][w0] -> A[0] (padded rows) and, for training, its transpose
int ingest(slp_segment* s, const void* X, int batch, bool with_transpose, hipStream_t st) {
  HIP_TRY(launch_copy_transpose(s->dtype, X, s->widths[0], batch, s->widths[0], s->A[0], s->ldw[0],
                                with_transpose ? s->AT[0] : nullptr, s->ldb, 1, nullptr, 0, st));
  return SLP_OK;
}

// Whether the cross-entropy is formed in the launch of the last layer's forward product.  (With one layer that launch would have the input's
// copies to make.)
bool xent_in_product(const slp_segment* s, int batch) {
  return s->loss == SLP_SOFTMAX_XENT && s->L > 1 && logits_fit(s->dtype, batch, s->widths[s->L], s->widths[s->L - 1]);
}

// Launches of a training step whose products are all small (one stream, no events); 0 for any other step.
int direct_launches(const slp_segment* s, const void* X, int batch);

// Whether the first layer's product can read the caller's dense input itself: a small layer whose input rows start on 16-byte
// boundaries.  The copies the rest of the step needs are then made in the same launch.
bool reads_input(const slp_segment* s, const void* X, int batch) {
  return product_is_small(s->dtype, EPI_FWD, batch, s->widths[1]) && (size_t)s->widths[0] * esize(s) % 16 == 0 && ((uintptr_t)X & 15) == 0;
}

int direct_launches(const slp_segment* s, const void* X, int batch) {
  for (int l = 1; l <= s->L; ++l)
    if (!product_is_small(s->dtype, EPI_FWD, batch, s->widths[l]) || !product_is_small(s->dtype, EPI_WGRAD_UPDATE, s->widths[l], s->widths[l - 1]) ||
        (l > 1 && !product_is_small(s->dtype, EPI_DGRAD, batch, s->widths[l - 1])))
      return 0;
  // ingest unless it rides along, forward, cross-entropy, data gradients (weight gradients ride along), the last weight gradients
  return (reads_input(s, X, batch) ? 0 : 1) + s->L + (s->loss == SLP_MSE_SIL || xent_in_product(s, batch) ? 0 : xent_launch_count(s->dtype, s->widths[s->L])) + (s->L - 1) + 1;
}

// The layers s + 1 .. L of a forward-only pass that go through one launch_chain, as s; L where there is no such run of two or more.  All of
// them are narrow, their products of the kind that sums in the chain's order, and the strips of the batch fit the chip at once (float32
// 64-64-64-64 at 8000 rows, two rounds: 10.3 us a pass in a launch each, 10.7 in one).
int chain_from(const slp_segment* s, int batch) {
  int from = s->L;
  if (batch > (s->dtype == SLP_BF16 ? 8192 : 4096)) return from;
  for (int l = s->L; l >= 1 && s->L - l < kChainLayers; --l) {
    const int N = s->widths[l], K = s->widths[l - 1];
    if (N > kChainWidth || K > kChainWidth || !product_is_small(s->dtype, EPI_FWD, batch, N) || small_tile(s->dtype, batch, N) >= 64) break;
    if (s->L - l >= 1) from = l - 1;
  }
  return from;
}

struct Forward {
  bool training;
  const void* X;            // the caller's input, dense
  const void* x_direct;     // large layers of a forward-only pass: X itself is the first layer's operand ...
  void* out_direct;         // ... and the caller's dense output buffer the last layer's result (their rows are aligned)
  void* out;                // forward-only: the caller's output buffer
  bool keeps_input;         // whether nothing is written to X before the last launch that could read it has ended, of one launch a layer
  bool apart;               // forward-only: the same of any number of layers a launch
  const OutJob* last;       // training: the gradient of the output rides along with a small last layer (neither table nor ext: cross-entropy)
  bool wait_by_layer;       // training: each layer's launches follow its update of the step before (see settle_step)
};

// What a layer's forward product waits for where settle_step left the wait to it.
int settle_layer(slp_segment* seg, int l, hipStream_t st) {
  if (l == seg->L && seg->paced) {       // (the last of them: see settle)
    HIP_TRY(launch_hurry(seg->hurry, 1, st));
    seg->paced = false;
  }
  HIP_TRY(hipStreamWaitEvent(st, seg->ev_update[l - 1], 0));
  return SLP_OK;
}

// Ingest and all layers.  *out_done: the last layer wrote f.out itself; *last_done: it formed the output's gradient.
int forward_layers(slp_segment* s, int batch, const Forward& f, hipStream_t st, bool* out_done, bool* last_done) {
  const bool direct = !f.x_direct && f.keeps_input && reads_input(s, f.X, batch);
  if (!f.x_direct && !direct) {
    int rc = ingest(s, f.X, batch, f.training, st);
    if (rc) return rc;
  }
  int from = f.training ? s->L : chain_from(s, batch);
  if (from == 0 && !f.apart) from = s->L;
  for (int l = 1; l <= from; ++l) {
    const Layer& ly = s->layers[l - 1];
    GemmArgs g{};
    g.A = s->A[l - 1]; g.lda = s->ldw[l - 1];
    if (l == 1 && (f.x_direct || direct)) { g.A = f.X; g.lda = s->widths[0]; }
    g.B = ly.Wop;      g.ldb = ly.ldk;
    g.M = batch; g.N = ly.N; g.K = ly.K;
    g.C = s->A[l]; g.ldc = s->ldw[l];
    if (l == s->L && f.out_direct) { g.C = f.out_direct; g.ldc = s->widths[l]; }
    g.CT = (f.training && l < s->L) ? s->AT[l] : nullptr; g.ldct = s->ldb;
    g.bits_out = (f.training && l < s->L) ? s->bits[l] : nullptr; g.ldbits = s->ldbits;
    g.bias = ly.b; g.relu = relu_on(s, l) ? 1 : 0;
    int rc = f.wait_by_layer ? settle_layer(s, l, st) : SLP_OK;
    if (rc) return rc;
    if (l == s->L && f.last && !f.last->table && !f.last->ext && xent_in_product(s, batch)) {
      rc = run_logits(s, g, *f.last, st);
      *last_done = true;
    } else if (product_is_small(s->dtype, EPI_FWD, g.M, g.N)) {
      SmallGroup gr{};
      gr.n = 1; gr.epi[0] = EPI_FWD;
      if (l == 1 && direct) {
        const int rows_t = (batch + 7) & ~7;
        gr.has_copy = true;
        gr.copy = CopyJob{f.X, s->widths[0], batch, s->widths[0], s->A[0], s->ldw[0], f.training ? s->AT[0] : nullptr, s->ldb, rows_t};
      }
      if (l == s->L && f.out && f.out != g.C) { g.C2 = f.out; g.ldc2 = s->widths[l]; *out_done = true; }
      if (l == s->L && f.last && (f.last->table || f.last->ext)) { gr.epi[0] = EPI_FWD_OUT; gr.out = *f.last; *last_done = true; }
      gr.g[0] = g;
      rc = run_group(s, gr, st);
    } else {
      rc = run_gemm(s, EPI_FWD, g, st);
    }
    if (rc) return rc;
  }
  if (from == s->L) return SLP_OK;
  ChainLaunch c{};
  const bool from_caller = from == 0 && (f.x_direct || direct);
  c.X = from_caller ? f.X : s->A[from]; c.ldx = from_caller ? s->widths[0] : s->ldw[from];
  c.K0 = s->widths[from]; c.M = batch; c.layers = s->L - from;
  c.relu_last = relu_on(s, s->L) ? 1 : 0;
  for (int i = 0; i < c.layers; ++i) {
    const int l = from + 1 + i;
    const Layer& ly = s->layers[l - 1];
    c.layer[i] = ChainLayer{ly.Wop, ly.b, l == s->L && f.out_direct ? nullptr : s->A[l], ly.N, ly.ldk, s->ldw[l]};
  }
  c.out = f.out;
  *out_done = true;
  if (from == 0 && direct) { c.copy = s->A[0]; c.ldcopy = s->ldw[0]; }
  return run_chain(s, c, st);
}

// Forward pass of a training step with the loss and dZ_L (row-major for the data gradient, transposed -- with_transpose --
// for the weight gradient).  *sum: the loss's partial sums, still to be added up.
int forward_and_loss(slp_segment* seg, const void* X, const int32_t* targets, int batch, bool with_transpose, float* loss_out,
                     bool wait_by_layer, SumJob* sum, hipStream_t st) {
  const int L = seg->L, D = seg->widths[L];
  bool out_done = false, last_done = false;
  OutJob oj{};
  const bool mse = seg->loss == SLP_MSE_SIL;
  oj.y = targets; oj.table = seg->table; oj.classes = seg->classes;
  oj.scale = mse ? (float)(2.0 / ((double)batch * (double)D)) : (float)(1.0 / (double)batch);
  oj.partials = seg->partials; oj.bad_ids = seg->bad_ids;
  oj.dZ = seg->dZ[L]; oj.lddz = seg->ldw[L]; oj.dZT = mse || with_transpose ? seg->dZT[L] : nullptr; oj.lddzt = seg->ldb;
  int rc = forward_layers(seg, batch, Forward{true, X, nullptr, nullptr, nullptr, true, true, &oj, wait_by_layer}, st, &out_done, &last_done);
  if (rc) return rc;
  *sum = SumJob{seg->partials, 0, 0.0, seg->loss_dev, loss_out};
  if (mse) {
    sum->scale = 1.0 / ((double)batch * D);
    sum->n = last_done ? small_tile_count(seg->dtype, batch, D) : mse_partial_count(batch, D);
    if (!last_done)
      HIP_TRY(launch_mse_loss_grad(seg->dtype, seg->A[L], seg->ldw[L], targets, seg->table, seg->classes, batch, D,
                                   relu_on(seg, L) ? 1 : 0, seg->dZ[L], seg->dZT[L], seg->ldb, seg->partials, seg->bad_ids, st));
  } else {
    sum->scale = 1.0 / (double)batch;
    sum->n = batch;
    if (!last_done)
      HIP_TRY(launch_xent_loss_grad(seg->dtype, seg->A[L], seg->ldw[L], targets, batch, D, relu_on(seg, L) ? 1 : 0,
                                    seg->dZ[L], with_transpose ? seg->dZT[L] : nullptr, seg->ldb, seg->partials, seg->bad_ids, st));
  }
  return SLP_OK;
}

// dZ_{l-1} = (dZ_l W_l) * [A_{l-1} > 0]; for l = 1 the result is the gradient w.r.t. the segment input (no mask)
GemmArgs data_gradient(slp_segment* seg, int l, int batch) {
  Layer& ly = seg->layers[l - 1];
  GemmArgs g{};
  g.A = seg->dZ[l]; g.lda = seg->ldw[l];
  g.B = ly.WT;      g.ldb = ly.ldn;
  g.M = batch; g.N = ly.K; g.K = ly.N;
  g.C = seg->dZ[l - 1]; g.ldc = seg->ldw[l - 1];
  g.CT = l > 1 ? seg->dZT[l - 1] : nullptr; g.ldct = seg->ldb;
  g.maskT = l > 1 ? seg->AT[l - 1] : nullptr; g.ldmask = seg->ldb;
  g.bits = l > 1 ? seg->bits[l - 1] : nullptr; g.ldbits = seg->ldbits;
  return g;
}

// Whether the caller asked for the optimiser step of this layer inside its weight-gradient product.
bool update_is_fused(const slp_segment* s, const Layer& ly) { return s->fused_update && (long)ly.N * ly.K <= s->fused_max_params; }

// Whether the update of a large layer goes into the launch of its weight-gradient product (launch_pair).  There the gradient is not read
// back and the update's streams run beside other tiles' products; but a product on 256x256 tiles is faster from some length of the batch
// on, and with it an update that runs beside the next products.  Microseconds a step, update apart / in the product's launch:
//   bf16      784-2048-2048-2048, 256 rows 114 / 103, 1600 206 / 173, 2048 219 / 197; 4096 wide, two layers, 1700 447 / 409, 2048 460 / 445, three,
//             256 346 / 296; 5000 wide, three, 1800 1210 / 1137, 2048 1424 / 1278; 6144 wide, three, 1536 1637 / 1464, 2048 1814 / 1718; 8192 wide,
//             two, 1700 1542 / 1435, 2048 1632 / 1575; 16384 wide, two, 512 3076 / 2081, 1700 6117 / 5598, 2048 6498 / 6138
//   beyond    784-2048-2048-2048, 2300 279 / 250, 4096 338 / 321; 4096 wide, three, 2300 993 / 943, 2600 1003 / 1026, 4096 1042 / 1123; 8192
//             wide, three, 2300 3234 / 3196, 2600 3265 / 3321, 4096 3891 / 4136; 16384 wide, two, 2300 7624 / 7156, 3000 8097 / 8234, 4096 9775 /
//             10591
//   float32   784-2048-2048-2048, 300 rows 298 / 258, 1024 531 / 515, 4096 1887 / 1808, 6000 2841 / 3003; 3000 wide, two layers, 1024 936 / 818,
//             4096 3409 / 3119, 6000 6495 / 6129; 4096 wide, two, 300 722 / 640, 4096 5029 / 4937, 6000 8727 / 8731; 6144 wide, two, 4096 14527 / 13068
// A weight gradient that is whole rounds of 256x256 tiles wastes nothing on them, and from seven rows of such tiles on the data gradients of wide
// layers take them too and have no launch in common with an update: there the update is faster apart as long as the products of two
// layers are still to come, for it to run beside.  All apart / all in the product / the third layer and those above it apart:
//   4096 wide three layers, 1100 rows - / 574 / 611, 1600 - / 651 / 664, 2048 744 / 767 / 762, four, 1600 - / 923 / 898, 2048 1014 / 1059 / 1035, six, 2048
//             1537 / 1623 / 1558; 8192 wide, three, 1500 - / 2457 / 2510, 1600 - / 2160 / 2134, 2048 2465 / 2463 / 2445, five, 1700 3819 / 3859 / 3750, 2048
//             4102 / 4246 / 4074; 784-8192-8192-8192-8192, 1700 2502 / 2519 / 2448; 12288 wide, three, 1600 - / 5099 / 5116, 1900 5660 / 5561 / 5462;
//             16384 wide, four, 2048 12882 / 13018 / 12753; the second layer apart as well: 784-8192-8192-8192, 2048 1924 for 1830
// With the join left to a later call a product in its own stream, beside the others (two such segments in turns, a step of both):
//   bf16      784-2048-2048-2048, 256 rows 254 / 202, 1024 355 / 306; 8192 wide, two layers, 512 1895 / 1671, 2048 2812 / 3100; 4096 wide, 2048
//             1505 / 1651;   float32 784-2048-2048-2048, 512 635 / 598; 4096 wide, 1024 2719 / 2727; 2048 wide, 2048 2267 / 2292
// Where the caller asked for it in any case (slp_segment_set_fused_update), a step with every product on its own tiles / in launch_pair:
//   bf16      784-4096, 512 rows 41 / 32, 4096 97.6 / 94.9, 8192 186.2 / 187.1; 784-2048-2048-2048, 4096 358 / 307, 6000 526 / 489;
//             1024-4096-1024-4096, 4096 419 / 393, 6000 615 / 621, 8192 760 / 797; 8192-8192, 512 579 / 311, 4096 1217 / 1115, 8192 1970 / 2050
//   float32   784-4096, 512 rows 85.5 / 75.8, 4096 510 / 499, 6000 859 / 845; 784-2048-2048-2048, 4096 1848 / 1798, 6000 2961 / 2985;
//             1024-4096-1024, 4096 1362 / 1323, 6000 2358 / 2319
bool update_in_product(const slp_segment* s, int l, int batch, bool defer) {
  const Layer& ly = s->layers[l - 1];
  const bool b16 = s->dtype == SLP_BF16;
  if (update_is_fused(s, ly)) return batch <= 4096;
  if (defer) return batch < (b16 ? 1400 : 640);
  if (b16 && batch > 1536 && l > 2 && product_fills_rounds(ly.N, ly.K)) return false;
  return batch <= (b16 ? 2048 : 4096);
}

// Makes `st` wait for updates a previous step left running on the side stream (deferred join).  The flag stays set
// until the next step replaces the event (or the host has waited): every stream that touches the handle in between
// gets the wait, not only the first one.
int settle(slp_segment* seg, hipStream_t st) {
  if (!seg->join_pending) return SLP_OK;
  if (st) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing(st, &cap));
    if (cap != hipStreamCaptureStatusNone)
      return fail(SLP_ERR_STATE, "updates of an overlapped step are still pending and a stream that is being captured cannot "
                                 "wait for them: call slp_segment_set_overlap(seg, 0) before the capture");
  }
  if (seg->paced) {     // when `st` gets here nothing of it runs beside the updates any more: no reason to pace them for it
    HIP_TRY(launch_hurry(seg->hurry, 1, st));
    seg->paced = false;
  }
  HIP_TRY(hipStreamWaitEvent(st, seg->ev_join, 0));
  return SLP_OK;
}

// The same for a step.  Where the updates came in the order of the layers, the step only needs each layer's when its forward pass gets
// there (*by_layer), and the tail of them runs beside the first products; what it needs at once, in whichever stream it is, is that the
// products of the step before have ended.  With graphs on, whose steps hold no such waits, it is the whole wait.
// A step of fewer rows than the pending one has less to run beside paced updates than they were paced for and raises the flag at once, not where
// it waits for the last of them: one handle of 784-16384-16384-16384, 8192 rows and 4096 in turns 15248 -> 15098 us a step, 8192 and 2048
// 13419 -> 13263; two handles in turns equal.
int settle_step(slp_segment* seg, int batch, hipStream_t st, bool* by_layer) {
  if (seg->join_pending && seg->pending_by_layer && !seg->use_graph) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (st) HIP_TRY(hipStreamIsCapturing(st, &cap));
    *by_layer = cap == hipStreamCaptureStatusNone;
  }
  if (!*by_layer) return settle(seg, st);
  HIP_TRY(hipStreamWaitEvent(st, seg->ev_fork[seg->L - 1], 0));      // (recorded behind the last of them)
  if (seg->paced && batch < seg->pending_batch) {
    HIP_TRY(launch_hurry(seg->hurry, 1, st));
    seg->paced = false;
  }
  return SLP_OK;
}

// The same on the host.  The pauses of paced updates are sat through: there is no stream at hand here to raise the flag on that
// is not behind work of the caller's.
int settle_on_host(slp_segment* seg) {
  if (!seg->join_pending) return SLP_OK;
  HIP_TRY(hipStreamSynchronize(seg->side));
  seg->join_pending = seg->paced = false;
  return SLP_OK;
}

// Weight updates of large layers that run on the side stream, beside the next matrix products, are held to one workgroup
// per compute unit (256, 512 and 128 were tried: 256 is best, -2 % per step on the comparison and deep configurations).
constexpr int kSideUpdateWorkgroups = 256;
// slp_segment_set_fused_update(seg, 2): layers up to this many weights take the update inside their weight-gradient product at any batch
// and do without a stored gradient.  Part of the interface: it says which gradients can be read back.
constexpr long kFusedAutoMaxWeights = 1L << 22;

constexpr size_t kMemoryCache = (size_t)256 << 20;
constexpr long kByLayerWeights = 1L << 26;       // (see backward_and_update)

// Backward and update, last layer first; the data gradient of layer l reads W_l before it is updated.
// Small layers: the weight gradient's product always applies the update in its epilogue (and stores the gradient as well, unless
// the fused update is on), and it waits for company: the product of layer l + 1 goes into one launch with the data gradient of
// layer l, which does not read what it writes, or with the weight gradient of layer l at the end; the bias gradients ride
// along, and `sum` with the first such launch.  A step of 784-128-64 is 4 launches instead of 10 that way.
// Larger layers whose update is in their product's launch (update_in_product) do the same in launch_pair, also with one layer small
// and the other not; but a small float32 data gradient stays by itself: on 128 columns a tile it has too few tiles for its products
// (784-2048-2048-2048, 256 rows: 336 us a step with it, 275 without).
int backward_and_update(slp_segment* seg, int batch, const SumJob* sum, hipStream_t st) {
  // a join cannot be left to a later call while the launches are being captured into a graph
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (seg->defer_join && st) HIP_TRY(hipStreamIsCapturing(st, &cap));
  const bool defer = seg->defer_join && cap == hipStreamCaptureStatusNone;
  bool forked = false;           // whether anything of this step went to the side stream
  auto fork = [&](int l) -> int {        // what goes to the side stream from here on follows what layer l has queued
    HIP_TRY(hipEventRecord(seg->ev_fork[l - 1], st));
    HIP_TRY(hipStreamWaitEvent(seg->side, seg->ev_fork[l - 1], 0));
    forked = true;
    return SLP_OK;
  };
  // What a step touches comes round again with the next one: from the memory-side cache if all of it fits, else past the caches, so
  // that the weights' copies and the activations, which this step reads again, stay there.  Microseconds a step, kept / streamed:
  // bf16, three layers 2048 wide (0.2 GB) 111 / 121, 2304 (0.26 GB) 170 / 166, 2560 (0.32 GB) 211 / 191, 3072 295 / 235, two layers 2560
  // wide (0.22 GB) 116 / 127; float32, three layers 2048 wide 279 / 292, 2560 400 / 395.
  const bool resident = seg->param_bytes + seg->work_bytes <= kMemoryCache;
  // With the join left to a later call and every layer's update apart, the data gradients come first and the weight gradients in the order
  // of the layers, so that the updates end in the order in which the next step needs them and the tail runs beside its first products
  // (settle_step), where the first layer's was waited for with nothing beside it.  From a layer of 8192x8192 on: smaller ones' updates are
  // as long as the products beside them, and spread over all of the backward pass they cost other segments less.  bf16, microseconds,
  // that order / this one, a step of one handle and of two in turns: 784-16384-16384-16384 8192 rows 19953 / 19432 and 37996 / 37972,
  // 784-16384-16384 4096 rows 6722 / 6026 and 11046 / 10952, 8192 wide, three layers, 4096 rows 4337 / 4024 and 7281 / 7244, 2048 rows
  // 2407 / 2309 and 4440 / 4435; 4096 wide, three layers, 4096 rows 926 / 908 and 1797 / 1809, 3000 rows 1019 / 1010 and 2011 / 2046.
  bool by_layer = defer && seg->dtype == SLP_BF16;
  long largest = 0;
  for (int l = 1; l <= seg->L && by_layer; ++l) {
    const Layer& ly = seg->layers[l - 1];
    largest = std::max(largest, (long)ly.N * ly.K);
    by_layer = !product_is_small(seg->dtype, EPI_WGRAD_UPDATE, ly.N, ly.K) && !update_is_fused(seg, ly) && !update_in_product(seg, l, batch, defer);
  }
  by_layer = by_layer && largest >= kByLayerWeights;
  // With the join left to a later call the update's tail has the caller's next work to hide behind, and the update can
  // be paced so that its loads fit beside the products' (see sgd_update_strided_kernel).  How long it may take scales
  // with the batch (the products beside it do): nothing up to 2048 rows, 8 units at 4096, capped at 14 from 5632 on --
  // measured: comparison configuration (8192 rows) best at 10-16 units, deep configuration run serially (4096) at 8-14,
  // wide configuration (1024) 18 % slower with any pause.  In the order of the layers an update has about one product's time until the
  // next step needs it, and less of a pause is best for one handle: 8192 wide, three layers, 4096 rows 4260 us a step with 8 units, 4144 with
  // 2 and with none; 16384 wide, 8192 rows 20515 with 13, 20585 with 14; 8192 wide, two layers, 5632 rows 3971 with 14, 3482 with 6.  Two
  // handles in turns want some of it from shorter batches on.  A step of both, updates in the old order / in this one without a pause / as here:
  // 8192 wide, two layers, 2304 rows 3844 / 3910 / 3858, 2700 4007 / 4058 / 3989, 3000 4068 / 4125 / 4050; 784-16384-16384, 2048 rows 6767 / 6787
  // / 6658, 2700 8517 / 8666 / 8539, 3000 8777 / 8972 / 8788; 784-8192-8192-8192-8192, 2048 rows 5125 / 5086 / 5009, 3300 7527 / 7576 / 7526.
  // What is still slower in this order: 8192 wide, three layers, 1500 rows 2764 / 2804, 1800 2480 / 2506, two handles 3000 rows 6360 / 6432.
  const int by_layer_pause = batch < 1792 ? 0 : batch < 2560 ? 1 : std::max(2, (batch - 3072) / 384);
  const int pause = !defer ? 0 : std::min(14, by_layer ? by_layer_pause : std::max(0, (batch - 2048) / 256));
  if (pause > 0) HIP_TRY(launch_hurry(seg->hurry, 0, st));
  while (by_layer && (int)seg->ev_update.size() < seg->L) {      // (the first such step of a handle)
    hipEvent_t e = nullptr;
    HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    seg->ev_update.push_back(e);
  }
  for (int l = seg->L; by_layer && l > 1; --l) {
    const int rc = run_gemm(seg, EPI_DGRAD, data_gradient(seg, l, batch), st);
    if (rc) return rc;
  }
  SmallGroup pending{};                  // products waiting for company
  bool pending_small = true;             // whether they are for launch_small_group or for launch_pair ...
  bool pending_pairs = false;            // ... or could be for either
  auto flush = [&]() -> int {
    if (!pending.n) return SLP_OK;
    if (sum) {
      pending.has_sum = true;
      pending.sum = *sum;
      sum = nullptr;
    }
    pending.resident = resident;
    const int rc = run_group(seg, pending, st, pending_small);
    pending = SmallGroup{};
    return rc;
  };
  for (int i = 0; i < seg->L; ++i) {
    const int l = by_layer ? i + 1 : seg->L - i;
    Layer& ly = seg->layers[l - 1];
    if (l > 1 && !by_layer) {
      GemmArgs d = data_gradient(seg, l, batch);
      const bool small = product_is_small(seg->dtype, EPI_DGRAD, d.M, d.N);
      const bool pairs = pending.n && pending_pairs && !(small && (pending_small || seg->dtype == SLP_F32)) && product_can_pair(seg->dtype, EPI_DGRAD, d.M, d.N);
      int rc = SLP_OK;
      if (pending.n && !pairs && (!small || !pending_small)) rc = flush();
      if (rc) return rc;
      if (pairs) {                       // the data gradient first: its tiles are the longer ones
        d.maskT = seg->A[l - 1]; d.ldmask = seg->ldw[l - 1];
        pending.g[1] = pending.g[0];
        pending.epi[1] = pending.epi[0];
        pending.g[0] = d;
        pending.epi[0] = EPI_DGRAD;
        pending.n = 2;
        pending_small = false;
        rc = flush();
      } else if (small) {
        pending.g[pending.n] = d;
        pending.epi[pending.n++] = EPI_DGRAD;
        pending_small = true;
        rc = flush();
      } else {
        rc = run_gemm(seg, EPI_DGRAD, d, st);
      }
      if (rc) return rc;
    }
    GemmArgs g{};
    g.A = seg->dZT[l];    g.lda = seg->ldb;
    g.B = seg->AT[l - 1]; g.ldb = seg->ldb;
    g.M = ly.N; g.N = ly.K; g.K = batch;
    g.Cf = ly.dW; g.ldc = ly.ldk;
    const bool fused = update_is_fused(seg, ly);
    const bool small = product_is_small(seg->dtype, EPI_WGRAD_UPDATE, g.M, g.N);
    if (fused) g.Cf = nullptr;
    if (small || fused || update_in_product(seg, l, batch, defer)) {
      // The data gradient of layer l read W_l^T before this product is queued.
      g.uW = ly.W32; g.uV = ly.vW; g.uW16 = ly.W16; g.uWT = ly.WT; g.ldwt = ly.ldn;
      g.lr = seg->lr; g.mu = seg->mu;
    }
    const BiasJob bias{seg->dZT[l], seg->ldb, ly.N, batch, ly.db, ly.b, ly.vb, seg->lr, seg->mu};
    const bool in_product = !small && update_in_product(seg, l, batch, defer);
    if (small || (in_product && (fused || !defer))) {      // waits for company
      const bool pairs = product_can_pair(seg->dtype, EPI_WGRAD_UPDATE, g.M, g.N) || !small;
      if (pending.n && pending_small != small && !(pending_pairs && pairs)) {
        int rc = flush();
        if (rc) return rc;
      }
      pending_small = small && (!pending.n || pending_small);
      pending_pairs = pairs;
      pending.g[pending.n] = g;
      pending.epi[pending.n++] = EPI_WGRAD_UPDATE;
      pending.bias[pending.n_bias++] = bias;
      continue;
    }
    int rc = flush();
    if (rc) return rc;
    if (in_product) {                      // left to a later call: beside what is still to come
      SmallGroup gr{};
      gr.n = gr.n_bias = 1;
      gr.g[0] = g; gr.epi[0] = EPI_WGRAD_UPDATE; gr.bias[0] = bias; gr.resident = resident;
      rc = fork(l);
      if (!rc) rc = run_group(seg, gr, seg->side, false);
      if (rc) return rc;
      continue;
    }
    rc = run_gemm(seg, fused ? EPI_WGRAD_UPDATE : EPI_WGRAD, g, st);
    if (rc) return rc;
    if (fused) {
      // What is left of the layer is its bias: one small launch, on the caller's stream (nothing worth a second stream).
      HIP_TRY(launch_layer_update(seg->dtype, nullptr, nullptr, nullptr, ly.N, 0, ly.ldk, nullptr, nullptr, ly.ldn, seg->dZT[l],
                                  seg->ldb, batch, ly.db, ly.b, ly.vb, seg->lr, seg->mu, st));
      continue;
    }
    // everything layer l still needs (bias gradient, both updates) reads dZ_l^T / dW_l, which are complete here, and writes
    // only layer l's parameters, which nothing below reads in this step; without a deferred join the first layer has nothing
    // left in this step to overlap with
    hipStream_t us = (defer || l > 1) ? seg->side : st;
    if (us != st) {
      rc = fork(l);
      if (rc) return rc;
    }
    // weights and bias in one launch, but for large layers beside products: there the bias part is a launch of its own first,
    // inside one launch its long reads of dZ^T slowed the products (measured 1 %)
    if ((size_t)ly.N * ly.K <= ((size_t)1 << 22) || us == st) {
      HIP_TRY(launch_layer_update(seg->dtype, ly.W32, ly.vW, ly.dW, ly.N, ly.K, ly.ldk, ly.W16, ly.WT, ly.ldn, seg->dZT[l],
                                  seg->ldb, batch, ly.db, ly.b, ly.vb, seg->lr, seg->mu, us));
    } else {
      HIP_TRY(launch_layer_update(seg->dtype, nullptr, nullptr, nullptr, ly.N, 0, ly.ldk, nullptr, nullptr, ly.ldn, seg->dZT[l],
                                  seg->ldb, batch, ly.db, ly.b, ly.vb, seg->lr, seg->mu, us));
      HIP_TRY(launch_update_beside(seg->dtype, ly.W32, ly.vW, ly.dW, ly.N, ly.K, ly.ldk, ly.W16, ly.WT, ly.ldn, seg->lr, seg->mu,
                                   kSideUpdateWorkgroups, pause, seg->hurry, us));
    }
    if (by_layer) HIP_TRY(hipEventRecord(seg->ev_update[l - 1], seg->side));
  }
  const int rc = flush();                // the last products; a fork and a join would cost more than they take
  if (rc) return rc;
  if (sum) HIP_TRY(launch_reduce_loss(sum->partials, sum->n, sum->scale, sum->out0, sum->out1, st));   // found no company
  if (forked) {     // join: later work on the caller's stream sees every update
    HIP_TRY(hipEventRecord(seg->ev_join, seg->side));
    if (!defer) HIP_TRY(hipStreamWaitEvent(st, seg->ev_join, 0));
  }
  seg->join_pending = defer && forked;
  seg->pending_by_layer = by_layer;
  seg->pending_batch = batch;
  seg->paced = seg->join_pending && pause > 0;
  return SLP_OK;
}

int refresh_copies(slp_segment* s, int layer, hipStream_t st) {
  Layer& ly = s->layers[layer];
  if (!ly.W16 && !ly.WT) return SLP_OK;
  HIP_TRY(launch_refresh_copies(s->dtype, ly.W32, ly.N, ly.K, ly.ldk, ly.W16, ly.WT, ly.ldn, st));
  return SLP_OK;
}

int copy_matrix(float* dense, float* padded, int rows, int cols, int ld, bool to_padded, int on_device, hipStream_t st) {
  const hipMemcpyKind kind = on_device ? hipMemcpyDeviceToDevice : (to_padded ? hipMemcpyHostToDevice : hipMemcpyDeviceToHost);
  if (to_padded)
    HIP_TRY(hipMemcpy2DAsync(padded, (size_t)ld * 4, dense, (size_t)cols * 4, (size_t)cols * 4, rows, kind, st));
  else
    HIP_TRY(hipMemcpy2DAsync(dense, (size_t)cols * 4, padded, (size_t)ld * 4, (size_t)cols * 4, rows, kind, st));
  return SLP_OK;
}

// Parameters up to this many floats go between device buffers in one launch of a kernel instead of a rectangle copy and a plain
// one of the runtime's, beyond it the two are equal.  Weights and bias, microseconds, runtime / kernel: 128 x 784 10.0 / 7.8, 2048 x 2048
// 9.9 / 7.7, 2048 x 2047 14.0 / 7.9, 4096 x 4096 21.8 / 20.9, 4096 x 4095 44.1 / 22.1, 8192 x 4096 42.8 / 43.3, 5792 x 5793 87.9 / 49.7.
constexpr long kSmallCopy = 1L << 25;
int exchange(slp_segment* s, int layer, float* W, float* b, int which, bool set, int on_device, hipStream_t st) {
  int rc = check_seg(s, true, !set);
  if (rc) return rc;
  if (layer < 0 || layer >= s->L) return fail(SLP_ERR_ARG, "layer %d out of range [0,%d)", layer, s->L);
  rc = settle(s, st);
  if (rc) return rc;
  Layer& ly = s->layers[layer];
  float* mats[3] = {ly.W32, ly.dW, ly.vW};
  float* vecs[3] = {ly.b, ly.db, ly.vb};
  if (W && which == 1 && update_is_fused(s, ly))
    return fail(SLP_ERR_STATE, "the weight gradient of layer %d is not stored: its update is fused into the product (slp_segment_set_fused_update)", layer);
  const bool small = on_device && (long)ly.N * ly.K <= kSmallCopy;
  if (small && (W || b)) {
    if (set) HIP_TRY(launch_copy_layer(W, ly.K, W ? mats[which] : nullptr, ly.ldk, ly.N, ly.K, b, vecs[which], st));
    else HIP_TRY(launch_copy_layer(W ? mats[which] : nullptr, ly.ldk, W, ly.K, ly.N, ly.K, b ? vecs[which] : nullptr, b, st));
  }
  if (W && !small) {
    rc = copy_matrix(W, mats[which], ly.N, ly.K, ly.ldk, set, on_device, st);
    if (rc) return rc;
  }
  if (b && !small) {
    const hipMemcpyKind kind = on_device ? hipMemcpyDeviceToDevice : (set ? hipMemcpyHostToDevice : hipMemcpyDeviceToHost);
    if (set) HIP_TRY(hipMemcpyAsync(vecs[which], b, (size_t)ly.N * 4, kind, st));
    else HIP_TRY(hipMemcpyAsync(b, vecs[which], (size_t)ly.N * 4, kind, st));
  }
  if (set && W) {
    rc = refresh_copies(s, layer, st);
    if (rc) return rc;
  }
  if (!on_device) HIP_TRY(hipStreamSynchronize(st));
  return SLP_OK;
}

}  // namespace

extern "C" {

const char* slp_last_error(void) { return g_err; }

int slp_make_synthetic_labels(uint64_t seed, int classes, int dim, int dist, float kappa, void* table, int dt,
                              slp_stream stream) {
  if (!table) return fail(SLP_ERR_ARG, "table is NULL");
  if (classes <= 0 || dim <= 0) return fail(SLP_ERR_ARG, "classes and dim must be positive (got %d, %d)", classes, dim);
  if (dist < SLP_UNIFORM01 || dist > SLP_BINARY_PM1) return fail(SLP_ERR_ARG, "unknown distribution %d", dist);
  if (dt != SLP_F32 && dt != SLP_BF16) return fail(SLP_ERR_ARG, "unknown dtype %d", dt);
  HIP_TRY(launch_make_labels(seed, classes, dim, dist, kappa, table, dt, (hipStream_t)stream));
  return SLP_OK;
}

int slp_make_segment_inputs(uint64_t seed, const float* table, int classes, const int32_t* y, int64_t first_sample,
                            int batch, int dim, float sigma, void* out, int dt, slp_stream stream) {
  if (!table || !y || !out) return fail(SLP_ERR_ARG, "table, y and out must not be NULL");
  if (classes <= 0 || dim <= 0 || batch <= 0 || first_sample < 0)
    return fail(SLP_ERR_ARG, "classes, dim, batch must be positive and first_sample non-negative");
  if (dt != SLP_F32 && dt != SLP_BF16) return fail(SLP_ERR_ARG, "unknown dtype %d", dt);
  HIP_TRY(launch_make_inputs(seed, table, classes, y, first_sample, batch, dim, sigma, out, dt, (hipStream_t)stream));
  return SLP_OK;
}

int slp_segment_create(const int* widths, int n_widths, int act, int loss, const slp_opts* opts, slp_segment** out) {
  if (!widths || !opts || !out) return fail(SLP_ERR_ARG, "widths, opts and out must not be NULL");
  *out = nullptr;
  if (n_widths < 2) return fail(SLP_ERR_ARG, "a segment needs at least one layer (n_widths = %d)", n_widths);
  if (n_widths > 65) return fail(SLP_ERR_ARG, "too many layers (%d)", n_widths - 1);
  for (int i = 0; i < n_widths; ++i)
    if (widths[i] <= 0 || widths[i] > (1 << 20)) return fail(SLP_ERR_ARG, "widths[%d] = %d is not in [1, 2^20]", i, widths[i]);
  if (act != SLP_RELU_ALL && act != SLP_RELU_HIDDEN_IDENTITY_LAST) return fail(SLP_ERR_ARG, "unknown activation rule %d", act);
  if (loss != SLP_MSE_SIL && loss != SLP_SOFTMAX_XENT) return fail(SLP_ERR_ARG, "unknown loss %d", loss);
  if (opts->dtype != SLP_F32 && opts->dtype != SLP_BF16) return fail(SLP_ERR_ARG, "unknown dtype %d", opts->dtype);
  if (opts->max_batch <= 0 || opts->max_batch > (1 << 24)) return fail(SLP_ERR_ARG, "max_batch = %d is not in [1, 2^24]", opts->max_batch);
  if (!(opts->lr >= 0.0f) || !(opts->momentum >= 0.0f && opts->momentum < 1.0f))
    return fail(SLP_ERR_ARG, "lr must be >= 0 and momentum in [0,1)");

  slp_segment* s = new slp_segment();
  s->L = n_widths - 1; s->act = act; s->loss = loss; s->dtype = opts->dtype; s->max_batch = opts->max_batch;
  s->ldb = internal_ld(opts->max_batch, opts->dtype == SLP_BF16 ? 2 : 4);
  s->lr = opts->lr; s->mu = opts->momentum;
  s->input_grad = opts->input_grad != 0;
  s->widths.assign(widths, widths + n_widths);
  for (int w : s->widths) s->ldw.push_back(internal_ld(w, opts->dtype == SLP_BF16 ? 2 : 4));
  const size_t es = esize(s);

  // every operand is addressed with 32-bit byte offsets below 2 GiB
  for (int l = 0; l <= s->L; ++l) {
    const size_t act_bytes = (size_t)std::max(s->ldb * (size_t)s->widths[l], (size_t)s->max_batch * s->ldw[l]) * es;
    if (act_bytes >= 0x80000000ull) {
      delete s;
      return fail(SLP_ERR_SHAPE, "activation of layer %d (%zu bytes) exceeds the 2 GiB operand limit", l, act_bytes);
    }
  }

  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align_up(bytes); return o; };
  for (int l = 0; l < s->L; ++l) {
    Layer ly{};
    ly.K = widths[l]; ly.N = widths[l + 1];
    ly.ldk = s->ldw[l]; ly.ldn = s->ldw[l + 1];
    const size_t wbytes = (size_t)ly.N * ly.ldk * 4;
    if (wbytes >= 0x80000000ull || (size_t)ly.K * ly.ldn * 4 >= 0x80000000ull) {
      delete s;
      return fail(SLP_ERR_SHAPE, "weight matrix of layer %d exceeds the 2 GiB operand limit", l);
    }
    ly.oW32 = take(wbytes); ly.ovW = take(wbytes); ly.odW = take(wbytes);
    ly.ob = take((size_t)ly.N * 4); ly.ovb = take((size_t)ly.N * 4); ly.odb = take((size_t)ly.N * 4);
    ly.oW16 = s->dtype == SLP_BF16 ? take((size_t)ly.N * ly.ldk * 2) : (size_t)-1;
    ly.oWT = (l > 0 || s->input_grad) ? take((size_t)ly.K * ly.ldn * es) : (size_t)-1;
    s->layers.push_back(ly);
  }
  s->param_bytes = off;

  off = 0;
  s->oA.assign(s->L + 1, (size_t)-1); s->oAT = s->oA; s->odZ = s->oA; s->odZT = s->oA; s->oBits = s->oA;
  s->ldbits = (s->max_batch + 127) / 128 * 4;
  for (int l = 0; l <= s->L; ++l) {
    s->oA[l] = take((size_t)s->max_batch * s->ldw[l] * es);
    if (l < s->L) s->oAT[l] = take((size_t)s->widths[l] * s->ldb * es);
    if (l >= 1 && l < s->L && s->dtype == SLP_BF16) s->oBits[l] = take((size_t)s->widths[l] * s->ldbits * 4);
    if (l == 0 && s->input_grad) s->odZ[0] = take((size_t)s->max_batch * s->ldw[0] * es);
    if (l >= 1) {
      // row-major dZ_l is the A operand of layer l's data gradient: needed for l >= 2, for the loss
      // kernels' output (l = L), and for l = 1 when the gradient w.r.t. the input is wanted
      if (l >= 2 || l == s->L || s->input_grad) s->odZ[l] = take((size_t)s->max_batch * s->ldw[l] * es);
      s->odZT[l] = take((size_t)s->widths[l] * s->ldb * es);
    }
  }
  // one per 64x64 tile of the output; small layers take smaller tiles, but never more than 1024 of them
  s->n_partials = loss == SLP_MSE_SIL ? std::max(mse_partial_count(s->max_batch, s->widths[s->L]), 1024) : s->max_batch;
  s->oPartials = take((size_t)s->n_partials * 4);
  s->oLoss = take(4);
  s->oBadIds = take(4);
  s->oHurry = take(4);
  s->work_bytes = off;

  s->side = nullptr; s->ev_join = nullptr;
  s->defer_join = false; s->join_pending = false; s->pending_by_layer = false; s->fused_update = false; s->fused_max_params = 0;
  s->bound = false; s->have_params = false; s->table = nullptr; s->classes = 0; s->last_batch = 0; s->prof = false;
  s->use_graph = false; s->graph_warm = false; s->graph_tick = 0; s->graph_misses = 0; s->graph_steps = 0;
  s->partials = nullptr; s->loss_dev = nullptr; s->bad_ids = nullptr;
  s->hurry = nullptr; s->paced = false;
  *out = s;
  return SLP_OK;
}

void slp_segment_destroy(slp_segment* seg) {
  if (!seg) return;
  for (auto& r : seg->prof_log) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
  for (auto e : seg->ev_pool) (void)hipEventDestroy(e);
  for (auto e : seg->ev_fork) (void)hipEventDestroy(e);
  for (auto e : seg->ev_update) (void)hipEventDestroy(e);
  if (seg->ev_join) (void)hipEventDestroy(seg->ev_join);
  drop_graphs(seg);
  if (seg->side) {
    (void)hipStreamSynchronize(seg->side);   // updates of a step with a deferred join may still be writing the caller's buffers
    (void)hipStreamDestroy(seg->side);
  }
  delete seg;
}

size_t slp_segment_param_bytes(const slp_segment* seg) { return seg ? seg->param_bytes : 0; }
size_t slp_segment_workspace_bytes(const slp_segment* seg) { return seg ? seg->work_bytes : 0; }

int slp_segment_bind(slp_segment* seg, void* params, size_t params_bytes, void* workspace, size_t workspace_bytes,
                     slp_stream stream) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  rc = settle_on_host(seg);    // the old buffers are still being written
  if (rc) return rc;
  if (!params || !workspace) return fail(SLP_ERR_ARG, "params and workspace must not be NULL");
  if (((uintptr_t)params | (uintptr_t)workspace) & (kAlign - 1)) return fail(SLP_ERR_ALLOC, "buffers must be 256-byte aligned");
  if (params_bytes < seg->param_bytes) return fail(SLP_ERR_ALLOC, "params buffer has %zu bytes, %zu needed", params_bytes, seg->param_bytes);
  if (workspace_bytes < seg->work_bytes) return fail(SLP_ERR_ALLOC, "workspace has %zu bytes, %zu needed", workspace_bytes, seg->work_bytes);
  hipStream_t st = (hipStream_t)stream;
  drop_graphs(seg);      // captured steps hold the old buffers' addresses
  seg->graph_warm = false;
  HIP_TRY(hipMemsetAsync(params, 0, seg->param_bytes, st));
  HIP_TRY(hipMemsetAsync(workspace, 0, seg->work_bytes, st));
  char* p = (char*)params;
  for (auto& ly : seg->layers) {
    ly.W32 = (float*)(p + ly.oW32); ly.vW = (float*)(p + ly.ovW); ly.dW = (float*)(p + ly.odW);
    ly.b = (float*)(p + ly.ob); ly.vb = (float*)(p + ly.ovb); ly.db = (float*)(p + ly.odb);
    ly.W16 = ly.oW16 == (size_t)-1 ? nullptr : (void*)(p + ly.oW16);
    ly.WT = ly.oWT == (size_t)-1 ? nullptr : (void*)(p + ly.oWT);
    ly.Wop = ly.W16 ? ly.W16 : (void*)ly.W32;
  }
  char* w = (char*)workspace;
  auto at = [&](size_t o) -> void* { return o == (size_t)-1 ? nullptr : (void*)(w + o); };
  seg->A.clear(); seg->AT.clear(); seg->dZ.clear(); seg->dZT.clear(); seg->bits.clear();
  for (int l = 0; l <= seg->L; ++l) {
    seg->A.push_back(at(seg->oA[l])); seg->AT.push_back(at(seg->oAT[l]));
    seg->dZ.push_back(at(seg->odZ[l])); seg->dZT.push_back(at(seg->odZT[l]));
    seg->bits.push_back((uint32_t*)at(seg->oBits[l]));
  }
  seg->partials = (float*)at(seg->oPartials);
  seg->loss_dev = (float*)at(seg->oLoss);
  seg->bad_ids = (unsigned*)at(seg->oBadIds);
  seg->hurry = (unsigned*)at(seg->oHurry);
  if (!seg->side) {     // host-side objects only; default priority
    HIP_TRY(hipStreamCreateWithFlags(&seg->side, hipStreamNonBlocking));
    HIP_TRY(hipEventCreateWithFlags(&seg->ev_join, hipEventDisableTiming));
    for (int l = 0; l < seg->L; ++l) {
      hipEvent_t e = nullptr;
      HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
      seg->ev_fork.push_back(e);
    }
  }
  seg->bound = true;
  seg->have_params = false;
  return SLP_OK;
}

int slp_segment_init(slp_segment* seg, uint64_t seed, slp_stream stream) {
  int rc = check_seg(seg, true, false);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  rc = settle(seg, st);
  if (rc) return rc;
  for (int l = 0; l < seg->L; ++l) {
    Layer& ly = seg->layers[l];
    HIP_TRY(launch_init_weights(seed, l, ly.W32, ly.N, ly.K, ly.ldk, ly.b, st));
    HIP_TRY(hipMemsetAsync(ly.vW, 0, (size_t)ly.N * ly.ldk * 4, st));
    HIP_TRY(hipMemsetAsync(ly.vb, 0, (size_t)ly.N * 4, st));
    rc = refresh_copies(seg, l, st);
    if (rc) return rc;
  }
  seg->have_params = true;
  return SLP_OK;
}

int slp_segment_set_params(slp_segment* seg, int layer, const float* W, const float* b, int on_device, slp_stream stream) {
  int rc = exchange(seg, layer, const_cast<float*>(W), const_cast<float*>(b), 0, true, on_device, (hipStream_t)stream);
  if (rc == SLP_OK) seg->have_params = true;
  return rc;
}
int slp_segment_get_params(slp_segment* seg, int layer, float* W, float* b, int on_device, slp_stream stream) {
  return exchange(seg, layer, W, b, 0, false, on_device, (hipStream_t)stream);
}
int slp_segment_get_grads(slp_segment* seg, int layer, float* dW, float* db, int on_device, slp_stream stream) {
  return exchange(seg, layer, dW, db, 1, false, on_device, (hipStream_t)stream);
}
int slp_segment_get_momentum(slp_segment* seg, int layer, float* vW, float* vb, int on_device, slp_stream stream) {
  return exchange(seg, layer, vW, vb, 2, false, on_device, (hipStream_t)stream);
}

int slp_segment_get_activation(slp_segment* seg, int layer, int kind, int batch, void* out, slp_stream stream) {
  int rc = check_seg(seg, true, false);
  if (rc) return rc;
  if (!out) return fail(SLP_ERR_ARG, "out is NULL");
  if (layer < 0 || layer > seg->L || (kind != 0 && kind != 1)) return fail(SLP_ERR_ARG, "layer %d / kind %d out of range", layer, kind);
  if (batch <= 0 || batch > seg->max_batch) return fail(SLP_ERR_SHAPE, "batch %d not in [1,%d]", batch, seg->max_batch);
  hipStream_t st = (hipStream_t)stream;
  rc = settle(seg, st);
  if (rc) return rc;
  const int w = seg->widths[layer];
  if (kind == 0) {
    HIP_TRY(launch_copy_transpose(seg->dtype, seg->A[layer], seg->ldw[layer], batch, w, out, w, nullptr, 0, 0, nullptr, 0, st));
  } else {
    if (layer < 1) return fail(SLP_ERR_ARG, "no gradient is formed for the segment input");
    if (seg->dZ[layer]) {
      HIP_TRY(launch_copy_transpose(seg->dtype, seg->dZ[layer], seg->ldw[layer], batch, w, out, w, nullptr, 0, 0, nullptr, 0, st));
    } else {   // only the transposed copy exists: transpose it back
      HIP_TRY(launch_copy_transpose(seg->dtype, seg->dZT[layer], seg->ldb, w, batch, nullptr, 0, out, w, 0, nullptr, 0, st));
    }
  }
  return SLP_OK;
}

int slp_segment_set_lr(slp_segment* seg, float lr, float momentum) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  if (!(lr >= 0.0f) || !(momentum >= 0.0f && momentum < 1.0f)) return fail(SLP_ERR_ARG, "lr must be >= 0 and momentum in [0,1)");
  seg->lr = lr; seg->mu = momentum;
  drop_graphs(seg);
  return SLP_OK;
}

int slp_segment_set_labels(slp_segment* seg, const float* table, int classes, int dim) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  if (seg->loss != SLP_MSE_SIL) return fail(SLP_ERR_STATE, "only a segment with the label-regression loss takes a label table");
  if (!table || classes <= 0) return fail(SLP_ERR_ARG, "table must not be NULL and classes positive");
  if (dim != seg->widths[seg->L]) return fail(SLP_ERR_SHAPE, "label dim %d != last width %d", dim, seg->widths[seg->L]);
  seg->table = table; seg->classes = classes;
  drop_graphs(seg);
  return SLP_OK;
}

int slp_segment_forward(slp_segment* seg, const void* X, int batch, void* out, slp_stream stream) {
  int rc = check_seg(seg, true, true);
  if (rc) return rc;
  if (!X || !out) return fail(SLP_ERR_ARG, "X and out must not be NULL");
  if (batch <= 0 || batch > seg->max_batch) return fail(SLP_ERR_SHAPE, "batch %d not in [1,%d]", batch, seg->max_batch);
  hipStream_t st = (hipStream_t)stream;
  rc = settle(seg, st);
  if (rc) return rc;
  // the stored-response pass over a whole dataset (Sec. 2) is this call in a loop: no activation is kept for a
  // backward pass, and dense caller buffers whose rows start on 16-byte boundaries are used in place
  const int w0 = seg->widths[0], w = seg->widths[seg->L];
  // One layer: its launch reads X and writes out, so where the two overlap X goes through the workspace.  (With more layers X has
  // been read before the launch that writes out begins.)
  const uintptr_t xa = (uintptr_t)X, oa = (uintptr_t)out;
  const bool apart = xa + (size_t)batch * w0 * esize(seg) <= oa || oa + (size_t)batch * w * esize(seg) <= xa;
  const bool keeps_input = seg->L > 1 || apart;
  const bool x_direct = keeps_input && w0 % kLdRows == 0 && (xa & 127) == 0;      // rows on cache-line boundaries, else the copy pays
  const bool out_direct = w % kLdAlign == 0 && ((uintptr_t)out & 15) == 0;
  bool out_done = false, last_done = false;
  rc = forward_layers(seg, batch, Forward{false, X, x_direct ? X : nullptr, out_direct ? out : nullptr, out, keeps_input, apart, nullptr, false}, st, &out_done,
                      &last_done);
  if (rc) return rc;
  if (!out_direct && !out_done)
    HIP_TRY(launch_copy_transpose(seg->dtype, seg->A[seg->L], seg->ldw[seg->L], batch, w, out, w, nullptr, 0, 0, nullptr, 0, st));
  seg->last_batch = batch;
  return SLP_OK;
}

int slp_segment_step(slp_segment* seg, const void* X, const int32_t* targets, int batch, float* loss_out, slp_stream stream) {
  int rc = check_seg(seg, true, true);
  if (rc) return rc;
  if (!X || !targets) return fail(SLP_ERR_ARG, "X and targets must not be NULL");
  if (batch <= 0 || batch > seg->max_batch) return fail(SLP_ERR_SHAPE, "batch %d not in [1,%d]", batch, seg->max_batch);
  if (seg->loss == SLP_MSE_SIL && !seg->table) return fail(SLP_ERR_STATE, "no label table bound: call slp_segment_set_labels first");
  hipStream_t st = (hipStream_t)stream;
  seg->last_batch = batch;
  bool by_layer = false;
  rc = settle_step(seg, batch, st, &by_layer);
  if (rc) return rc;

  auto launch_all = [&]() -> int {
    SumJob sum{};
    int r = forward_and_loss(seg, X, targets, batch, true, loss_out, by_layer, &sum, st);
    if (!r) r = backward_and_update(seg, batch, &sum, st);
    return r;
  };
  // Eager launches when graphs are off, when launches are being timed one by one, on the null stream (it
  // cannot be captured), and when the caller is capturing this stream already (the launches then go into
  // the caller's graph).  The first step of a handle is eager too, so that one-time kernel set-up is over
  // before anything is captured.
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (seg->use_graph && st) HIP_TRY(hipStreamIsCapturing(st, &cap));
  // A caller that never repeats a combination (a loop over more distinct batch buffers than the cache holds) would
  // pay a capture per step: after 2 x cache size misses in a row the handle goes back to eager launches until
  // slp_segment_set_graph is called again.
  const bool thrashing = seg->graph_misses > 2 * (int)kMaxStepGraphs;
  const int direct = seg->use_graph ? direct_launches(seg, X, batch) : 0;
  if (!seg->use_graph || thrashing || (direct > 0 && direct <= kDirectLaunches) || seg->prof || !st || cap != hipStreamCaptureStatusNone || !seg->graph_warm) {
    seg->graph_warm = true;
    return launch_all();
  }
  ++seg->graph_tick;
  for (auto& g : seg->graphs)
    if (g.X == X && g.targets == targets && g.batch == batch && g.loss_out == loss_out) {
      g.used = seg->graph_tick;
      seg->graph_misses = 0;
      HIP_TRY(hipGraphLaunch(g.exec, st));
      ++seg->graph_steps;
      return SLP_OK;
    }
  ++seg->graph_misses;
  HIP_TRY(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
  rc = launch_all();
  hipGraph_t graph = nullptr;
  hipError_t e = hipStreamEndCapture(st, &graph);      // always ended, so that the stream is usable after an error
  if (rc || e != hipSuccess) {
    if (graph) (void)hipGraphDestroy(graph);
    return rc ? rc : fail(SLP_ERR_DEVICE, "hipStreamEndCapture: %s", hipGetErrorString(e));
  }
  StepGraph sg{X, targets, batch, loss_out, nullptr, seg->graph_tick};
  e = hipGraphInstantiate(&sg.exec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) return fail(SLP_ERR_DEVICE, "hipGraphInstantiate: %s", hipGetErrorString(e));
  if (seg->graphs.size() >= kMaxStepGraphs) {          // evict the least recently used
    size_t v = 0;
    for (size_t i = 1; i < seg->graphs.size(); ++i)
      if (seg->graphs[i].used < seg->graphs[v].used) v = i;
    HIP_TRY(hipDeviceSynchronize());                   // its last replay may still be running
    (void)hipGraphExecDestroy(seg->graphs[v].exec);
    seg->graphs[v] = sg;
  } else {
    seg->graphs.push_back(sg);
  }
  HIP_TRY(hipGraphLaunch(sg.exec, st));
  ++seg->graph_steps;
  return SLP_OK;
}

int slp_segment_target_errors(slp_segment* seg, int64_t* count_out, slp_stream stream) {
  int rc = check_seg(seg, true, false);
  if (rc) return rc;
  if (!count_out) return fail(SLP_ERR_ARG, "count_out is NULL");
  hipStream_t st = (hipStream_t)stream;
  unsigned n = 0;
  HIP_TRY(hipMemcpyAsync(&n, seg->bad_ids, sizeof(n), hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  *count_out = (int64_t)n;
  return SLP_OK;
}

int slp_segment_set_graph(slp_segment* seg, int on) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  if (on) HIP_TRY(gemm_configure_all());
  seg->use_graph = on != 0;
  seg->graph_misses = 0;
  if (!seg->use_graph) drop_graphs(seg);
  return SLP_OK;
}

int slp_segment_graph_stats(const slp_segment* seg, int* captured, int64_t* replayed) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  if (captured) *captured = (int)seg->graphs.size();
  if (replayed) *replayed = seg->graph_steps;
  return SLP_OK;
}

int slp_segment_set_overlap(slp_segment* seg, int on) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  seg->defer_join = on != 0;
  return on ? SLP_OK : settle_on_host(seg);      // off: back to ordinary stream order, nothing is left running
}

int slp_segment_set_fused_update(slp_segment* seg, int on) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  if (on < 0) return fail(SLP_ERR_ARG, "slp_segment_set_fused_update: on must be >= 0 (got %d)", on);
  rc = settle_on_host(seg);            // updates of the other kind may still be running on the side stream
  if (rc) return rc;
  seg->fused_update = on != 0;
  seg->fused_max_params = on == 1 ? (1L << 62) : (on == 2 ? kFusedAutoMaxWeights : (long)on);
  drop_graphs(seg);                    // captured steps hold the other launch sequence
  return SLP_OK;
}

int slp_segment_join(slp_segment* seg, slp_stream stream) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  return settle(seg, (hipStream_t)stream);
}

int slp_segment_input_grad(slp_segment* seg, const void* X, const int32_t* targets, int batch, void* dX, float* loss_out,
                           slp_stream stream) {
  int rc = check_seg(seg, true, true);
  if (rc) return rc;
  if (!seg->input_grad) return fail(SLP_ERR_STATE, "segment was created without input_grad");
  if (!X || !targets || !dX) return fail(SLP_ERR_ARG, "X, targets and dX must not be NULL");
  if (batch <= 0 || batch > seg->max_batch) return fail(SLP_ERR_SHAPE, "batch %d not in [1,%d]", batch, seg->max_batch);
  if (seg->loss == SLP_MSE_SIL && !seg->table) return fail(SLP_ERR_STATE, "no label table bound: call slp_segment_set_labels first");
  hipStream_t st = (hipStream_t)stream;
  rc = settle(seg, st);
  if (rc) return rc;
  SumJob sum{};
  rc = forward_and_loss(seg, X, targets, batch, false, loss_out, false, &sum, st);
  if (rc) return rc;
  const int w0 = seg->widths[0];
  bool summed = false, dx_done = false;
  for (int l = seg->L; l >= 1; --l) {       // data gradients only, down to the input; parameters untouched
    GemmArgs d = data_gradient(seg, l, batch);
    if (product_is_small(seg->dtype, EPI_DGRAD, d.M, d.N)) {
      SmallGroup gr{};
      if (l == 1) { d.C2 = dX; d.ldc2 = w0; dx_done = true; }
      gr.g[0] = d; gr.epi[0] = EPI_DGRAD; gr.n = 1;
      if (!summed) { gr.has_sum = summed = true; gr.sum = sum; }
      rc = run_group(seg, gr, st);
    } else {
      rc = run_gemm(seg, EPI_DGRAD, d, st);
    }
    if (rc) return rc;
  }
  if (!summed) HIP_TRY(launch_reduce_loss(sum.partials, sum.n, sum.scale, sum.out0, sum.out1, st));
  if (!dx_done)
    HIP_TRY(launch_copy_transpose(seg->dtype, seg->dZ[0], seg->ldw[0], batch, w0, dX, w0, nullptr, 0, 0, nullptr, 0, st));
  seg->last_batch = batch;
  return SLP_OK;
}

int slp_segment_step_external(slp_segment* seg, const void* X, const void* dA_out, int batch, slp_stream stream) {
  int rc = check_seg(seg, true, true);
  if (rc) return rc;
  if (!X || !dA_out) return fail(SLP_ERR_ARG, "X and dA_out must not be NULL");
  if (batch <= 0 || batch > seg->max_batch) return fail(SLP_ERR_SHAPE, "batch %d not in [1,%d]", batch, seg->max_batch);
  hipStream_t st = (hipStream_t)stream;
  rc = settle(seg, st);
  if (rc) return rc;
  const int L = seg->L, D = seg->widths[L];
  // dZ_L = dA_out * [A_L > 0] (ReLU on the last layer) or dA_out, in both layouts
  OutJob oj{};
  oj.ext = dA_out;
  oj.dZ = seg->dZ[L]; oj.lddz = seg->ldw[L]; oj.dZT = seg->dZT[L]; oj.lddzt = seg->ldb;
  bool out_done = false, last_done = false;
  rc = forward_layers(seg, batch, Forward{true, X, nullptr, nullptr, nullptr, true, true, &oj, false}, st, &out_done, &last_done);
  if (rc) return rc;
  if (!last_done)
    HIP_TRY(launch_copy_transpose(seg->dtype, dA_out, D, batch, D, seg->dZ[L], seg->ldw[L], seg->dZT[L], seg->ldb, 1,
                                  relu_on(seg, L) ? seg->A[L] : nullptr, seg->ldw[L], st));
  rc = backward_and_update(seg, batch, nullptr, st);
  if (rc) return rc;
  seg->last_batch = batch;
  return SLP_OK;
}

int slp_count_correct(const void* logits, const int32_t* targets, int batch, int classes, int dt, void* scratch,
                      size_t scratch_bytes, int accumulate, int64_t* correct_out, slp_stream stream) {
  if (!logits || !targets || !scratch || !correct_out) return fail(SLP_ERR_ARG, "slp_count_correct: null pointer");
  if (batch <= 0 || classes <= 0) return fail(SLP_ERR_ARG, "slp_count_correct: batch and classes must be positive (got %d, %d)", batch, classes);
  if (dt != SLP_F32 && dt != SLP_BF16) return fail(SLP_ERR_ARG, "slp_count_correct: unknown dtype %d", dt);
  const size_t need = (size_t)count_partials(batch) * sizeof(int32_t);
  if (scratch_bytes < need || ((uintptr_t)scratch & 3))
    return fail(SLP_ERR_ALLOC, "slp_count_correct: scratch of %zu bytes (4-byte aligned) needed, %zu given", need, scratch_bytes);
  HIP_TRY(launch_count_correct(dt, logits, targets, batch, classes, (int32_t*)scratch, accumulate, (long long*)correct_out,
                               (hipStream_t)stream));
  return SLP_OK;
}

int slp_count_correct_static(const void* logits, const int32_t* targets, int batch, int classes, int dt, int accumulate,
                             int64_t* correct_out, slp_stream stream) {
  if (!logits || !targets || !correct_out) return fail(SLP_ERR_ARG, "slp_count_correct_static: null pointer");
  if (batch <= 0 || classes <= 0)
    return fail(SLP_ERR_ARG, "slp_count_correct_static: batch and classes must be positive (got %d, %d)", batch, classes);
  if (dt != SLP_F32 && dt != SLP_BF16) return fail(SLP_ERR_ARG, "slp_count_correct_static: unknown dtype %d", dt);
  static_assert(SLP_COUNT_STATIC_MAX_BATCH == 4 * kCountStaticPartials, "header limit and array size must agree");
  if (batch > SLP_COUNT_STATIC_MAX_BATCH)
    return fail(SLP_ERR_SHAPE, "slp_count_correct_static: batch %d exceeds the static scratch's limit of %d rows", batch,
                SLP_COUNT_STATIC_MAX_BATCH);
  int32_t* partials = nullptr;
  HIP_TRY(count_static_scratch(&partials));      // looked up once per device; never the array's name itself
  HIP_TRY(launch_count_correct(dt, logits, targets, batch, classes, partials, accumulate, (long long*)correct_out,
                               (hipStream_t)stream));
  return SLP_OK;
}

int slp_mean_loss(const float* losses, int n, float* mean_out, slp_stream stream) {
  if (!losses || !mean_out) return fail(SLP_ERR_ARG, "slp_mean_loss: null pointer");
  if (n <= 0) return fail(SLP_ERR_ARG, "slp_mean_loss: n must be positive (got %d)", n);
  HIP_TRY(launch_reduce_loss(losses, n, 1.0 / (double)n, mean_out, nullptr, (hipStream_t)stream));
  return SLP_OK;
}

int slp_segment_profile_enable(slp_segment* seg, int on) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  seg->prof = on != 0;
  // on > 1: create that many event pairs now, so that none is created between timed launches
  for (int i = (int)seg->ev_pool.size(); on > 1 && i < 2 * on; ++i) {
    hipEvent_t e = nullptr;
    HIP_TRY(hipEventCreate(&e));
    seg->ev_pool.push_back(e);
  }
  return SLP_OK;
}

int slp_segment_profile_read(slp_segment* seg, double* gemm_ms, int64_t* gemm_launches, double* gemm_flops) {
  int rc = check_seg(seg, false, false);
  if (rc) return rc;
  double ms = 0.0, fl = 0.0;
  int64_t n = 0;
  for (auto& r : seg->prof_log) {
    HIP_TRY(hipEventSynchronize(r.b));
    float t = 0.0f;
    HIP_TRY(hipEventElapsedTime(&t, r.a, r.b));
    ms += t; fl += r.flops; ++n;
    seg->ev_pool.push_back(r.a);
    seg->ev_pool.push_back(r.b);
  }
  seg->prof_log.clear();
  if (gemm_ms) *gemm_ms = ms;
  if (gemm_launches) *gemm_launches = n;
  if (gemm_flops) *gemm_flops = fl;
  return SLP_OK;
}

int slp_probe_mfma_rate(int dtype, int iters, void* scratch, size_t scratch_bytes, double* tflops, double* ms, slp_stream stream) {
  if (dtype != SLP_F32 && dtype != SLP_BF16) return fail(SLP_ERR_ARG, "slp_probe_mfma_rate: unknown dtype %d", dtype);
  if (iters <= 0 || iters > (1 << 24)) return fail(SLP_ERR_ARG, "slp_probe_mfma_rate: iters %d outside [1, 2^24]", iters);
  if (!scratch || !tflops) return fail(SLP_ERR_ARG, "slp_probe_mfma_rate: null scratch or result pointer");
  int dev = 0, cus = 0;
  HIP_TRY(hipGetDevice(&dev));
  HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const size_t per_wg = 512 * sizeof(float);
  if (scratch_bytes < per_wg * (size_t)cus)
    return fail(SLP_ERR_SHAPE, "slp_probe_mfma_rate: scratch of %zu bytes, %zu needed (%d compute units x 2048)", scratch_bytes,
                per_wg * (size_t)cus, cus);
  hipStream_t s = (hipStream_t)stream;
  hipEvent_t a = nullptr, b = nullptr;
  HIP_TRY(hipEventCreate(&a));
  HIP_TRY(hipEventCreate(&b));
  double fl = 0.0;
  hipError_t e = launch_mfma_probe(dtype, iters / 8 + 1, cus, (float*)scratch, &fl, s);   // warm-up: clocks settle
  if (e == hipSuccess) e = hipEventRecord(a, s);
  if (e == hipSuccess) e = launch_mfma_probe(dtype, iters, cus, (float*)scratch, &fl, s);
  if (e == hipSuccess) e = hipEventRecord(b, s);
  if (e == hipSuccess) e = hipEventSynchronize(b);
  float t = 0.0f;
  if (e == hipSuccess) e = hipEventElapsedTime(&t, a, b);
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (e != hipSuccess) return fail(SLP_ERR_DEVICE, "slp_probe_mfma_rate: %s", hipGetErrorString(e));
  *tflops = fl * cus * iters / (t * 1e-3) / 1e12;
  if (ms) *ms = t;
  return SLP_OK;
}

}  // extern "C"
