// Host side of the dense-tower C ABI (include/ctr_mlp.h): memory layout, the sequence of hand-written
// kernels of one training step (the bf16 matrix products of gemm_kernels.h with their fused epilogues, the
// element-wise kernels of mlp_kernels.h), the dense optimizer and its merge.
#include "../../include/ctr_mlp.h"
#include "../../include/ctr_sparse.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "common.h"
#include "gemm_kernels.h"
#include "mlp_kernels.h"

using namespace ctr;

namespace {

static_assert(CTR_MLP_MAX_HIDDEN + 1 <= COLSUM_MAX_JOBS, "a batch sum per hidden layer and one");
constexpr u32 MAX_WIDTH = 65536;
constexpr size_t GEMM_SCRATCH_MIN = (size_t)32 << 20;
static_assert(COLSUM_SLICES * MAX_WIDTH * sizeof(float) <= GEMM_SCRATCH_MIN, "room for the batch sums of one layer");
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
// Scratch for products whose contraction is split over several workgroups (gemm_kernels.h): room for
// four fp32 partial copies of the largest weight gradient, at least 32 MiB, at most 512 MiB.  A product
// that would need more is split less.
size_t gemm_scratch_bytes(const ctr_mlp_config* c) {
  size_t mx = 0;
  for (u32 l = 0; l < c->n_hidden; ++l)
    mx = std::max(mx, (size_t)(l == 0 ? c->in_dim : c->hidden[l - 1]) * c->hidden[l] * sizeof(float));
  return std::min<size_t>(std::max<size_t>(align256(4 * mx), GEMM_SCRATCH_MIN), (size_t)512 << 20);
}
inline u32 blocks_for(u64 threads) { return (u32)((threads + BLOCK - 1) / BLOCK); }

bool mlp_config_ok(const ctr_mlp_config* c) {
  if (!c) return false;
  if (c->in_dim == 0 || c->in_dim % 8 != 0) return false;
  if (c->n_hidden == 0 || c->n_hidden > CTR_MLP_MAX_HIDDEN) return false;
  for (u32 i = 0; i < c->n_hidden; ++i)
    if (c->hidden[i] == 0 || c->hidden[i] % 8 != 0 || c->hidden[i] > MAX_WIDTH) return false;
  if (c->n_replicas == 0 || c->n_replicas > 31) return false;
  if (c->kstep > 1) return false;
  if (!c->kstep && c->n_replicas != 1) return false;
  if (!(c->lr > 0.0f) || !(c->beta1 >= 0.0f && c->beta1 < 1.0f) || !(c->beta2 >= 0.0f && c->beta2 < 1.0f) ||
      !(c->eps > 0.0f))
    return false;
  return true;
}

void make_layout(const ctr_mlp_config* c, MlpLayout* L) {
  L->n_layers = c->n_hidden + 1;
  u64 off = 0;
  for (u32 l = 0; l < L->n_layers; ++l) {
    L->in[l] = l == 0 ? c->in_dim : c->hidden[l - 1];
    L->out[l] = l < c->n_hidden ? c->hidden[l] : 1;
    L->w_off[l] = off;
    off += (u64)L->in[l] * L->out[l] + L->out[l];
  }
  L->n_params = off;
}

struct MemLayout {
  u64 stride;  // elements between replicas (n_params rounded up to 128)
  size_t off_params, off_m, off_v, off_pb, off_vhat, total;
};

void mem_layout(const ctr_mlp_config* c, const MlpLayout& L, MemLayout* M) {
  M->stride = (L.n_params + 127) & ~(u64)127;
  const size_t W = c->n_replicas;
  size_t o = 0;
  M->off_params = o; o += align256(M->stride * W * sizeof(float));
  M->off_m = o; o += align256(M->stride * W * sizeof(float));
  M->off_v = o; o += align256(M->stride * W * sizeof(float));
  M->off_pb = o; o += align256(M->stride * W * sizeof(bf16_t));
  M->off_vhat = o;
  if (c->kstep) o += align256(M->stride * sizeof(float));
  M->total = o;
}

struct WsLayout {
  size_t off_h0, off_act[CTR_MLP_MAX_HIDDEN], off_dz, off_dlogit, off_lterm, off_grads, off_gemm,
      gemm_bytes, total;
};

void ws_layout(const ctr_mlp_config* c, const MlpLayout& L, u32 B, WsLayout* S) {
  const u32 last = c->hidden[c->n_hidden - 1];
  size_t o = 0;
  S->off_h0 = o; o += align256((size_t)B * c->in_dim * sizeof(bf16_t));
  for (u32 i = 0; i < c->n_hidden; ++i) {
    S->off_act[i] = o;
    o += align256((size_t)B * c->hidden[i] * sizeof(bf16_t));
  }
  S->off_dz = o; o += align256((size_t)B * last * sizeof(bf16_t));  // the other layers' dz take the place of act
  S->off_dlogit = o; o += align256((size_t)B * sizeof(float));
  S->off_lterm = o; o += align256((size_t)B * sizeof(double));
  S->off_grads = o; o += align256((size_t)L.n_params * sizeof(float));
  S->off_gemm = o; S->gemm_bytes = gemm_scratch_bytes(c);
  o += S->gemm_bytes;
  S->total = o;
}

inline int launch_status() { return hipGetLastError() == hipSuccess ? CTR_OK : CTR_E_DEVICE; }

}  // namespace

struct ctr_mlp {
  ctr_mlp_config cfg;
  MlpLayout L;
  MemLayout M;
  char* mem;
  float *params, *m, *v, *vhat;
  bf16_t* pb;
  u32 pend_mask;  // replicas whose last step was a merge step not merged yet
};

namespace {

// The three products of a hidden layer with row-major matrices, as C[M x N] = A B of gemm_kernels.h
// (which operand is stored with the contraction index contiguous differs from product to product):
//   forward          act[B x o]  = bf16(relu(H[B x i] W[i x o] + bias))     A = H (k-contiguous), B = W (n-contiguous)
//   weight gradient  dW[i x o]   = H^T[i x B] dZ[B x o]                     A = H (m-contiguous), B = dZ (n-contiguous)
//   input gradient   dH[B x i]   = dZ[B x o] W^T[o x i]                     A = dZ (k-contiguous), B = W (k-contiguous)
// The input gradient of a hidden layer goes straight through the ReLU of the layer below (mask = that
// layer's activation) and is stored as bf16; the first layer's is the gradient of the pooled input,
// stored as fp32 or bf16.
bool product_forward(const MlpLayout& L, u32 l, u32 B, const bf16_t* h, const bf16_t* w, const float* bias,
                     bf16_t* act, char* ws, const WsLayout& S, hipStream_t st) {
  GemmArgs g{};
  g.A = h; g.lda = L.in[l];
  g.B = w; g.ldb = L.out[l];
  g.M = B; g.N = L.out[l]; g.K = L.in[l];
  g.C16 = act; g.ldc = L.out[l];
  g.bias = bias;
  g.epilogue = EPI_BIAS_RELU_BF16;
  return gemm_enqueue(true, false, g, (float*)(ws + S.off_gemm), S.gemm_bytes, st) == hipSuccess;
}

GemmArgs weight_grad_args(const MlpLayout& L, u32 l, u32 B, const bf16_t* h, const bf16_t* dz, float* dw) {
  GemmArgs g{};
  g.A = h; g.lda = L.in[l];
  g.B = dz; g.ldb = L.out[l];
  g.M = L.in[l]; g.N = L.out[l]; g.K = B;
  g.C32 = dw; g.ldc = L.out[l];
  g.epilogue = EPI_F32;
  return g;
}

// exactly one of out32 / out16 / (mask, out16): fp32, bf16, or bf16 gated by the sign of `mask`
GemmArgs input_grad_args(const MlpLayout& L, u32 l, u32 B, const bf16_t* dz, const bf16_t* w, float* out32, bf16_t* out16,
                         const bf16_t* mask) {
  GemmArgs g{};
  g.A = dz; g.lda = L.out[l];
  g.B = w; g.ldb = L.out[l];
  g.M = B; g.N = L.in[l]; g.K = L.out[l];
  g.C32 = out32; g.C16 = out16; g.ldc = L.in[l];
  g.mask = mask;
  g.epilogue = out32 ? EPI_F32 : (mask ? EPI_RELU_MASK_BF16 : EPI_BF16);
  return g;
}

// How the backward pass of a step is launched, by its sizes.
// A layer whose two products take less time together than one after the other runs them in one launch (paired); its input
// gradient then has a place of its own instead of the activation's.  (One after the other is priced with the second launch of a
// split weight gradient, which kept sums do without.  in_place: the first layer's input gradient overlaps its input, which
// the weight gradient has to have read before.)  The partial sums of split weight gradients and of the sums over the batch stay
// where they are until the optimizer adds them (kept).  All that stands in the scratch of the products; where it does not
// fit, every product and every sum is finished by its own launches, in turn, but for the first layer's weight gradient, the
// last product of all: its partial sums have the scratch to themselves (first_kept), the sums over the batch then stand
// where its finished gradient would.
struct BackwardPlan {
  bool kept, first_kept, paired[CTR_MLP_MAX_HIDDEN];
  GemmPlan w[CTR_MLP_MAX_HIDDEN], i[CTR_MLP_MAX_HIDDEN];
  size_t off_w[CTR_MLP_MAX_HIDDEN], off_dz[CTR_MLP_MAX_HIDDEN], off_sums, off_rest;  // in the scratch
};

inline bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
  return (uintptr_t)a < (uintptr_t)b + b_bytes && (uintptr_t)b < (uintptr_t)a + a_bytes;
}

inline size_t split_bytes(const GemmPlan& p, u64 M, u64 N) { return p.n_split > 1 ? p.n_split * M * N * sizeof(float) : 0; }

void backward_plan(const MlpLayout& L, u32 B, size_t room, bool in_place, BackwardPlan* P) {
  const u32 hidden = L.n_layers - 1;
  size_t o = 0, rest = 0;
  u64 cols = L.in[hidden];
  for (u32 l = 0; l < hidden; ++l) {
    const u32 in = L.in[l], out = L.out[l];
    P->w[l] = gemm_plan(in, out, B, room);
    P->i[l] = gemm_plan(B, in, out, room);
    GemmPlan w, i;
    P->paired[l] = gemm_pair_plan(in, out, B, B, in, out, room, &w, &i) < P->w[l].cost + P->i[l].cost && !(in_place && l == 0);
    if (P->paired[l]) {
      P->w[l] = w;
      P->i[l] = i;
    }
    P->off_w[l] = o;
    o += align256(split_bytes(P->w[l], in, out));
    P->off_dz[l] = o;
    if (P->paired[l] && l > 0) o += align256((size_t)B * in * sizeof(bf16_t));
    rest = std::max(rest, split_bytes(P->i[l], B, in));
    cols += out;
  }
  P->off_sums = o;
  o += align256((size_t)COLSUM_SLICES * cols * sizeof(float));
  P->off_rest = o;
  P->kept = o + rest <= room;
  P->first_kept = false;
  if (P->kept) return;
  for (u32 l = 0; l < hidden; ++l) {
    P->paired[l] = false;
    P->w[l] = gemm_plan(L.in[l], L.out[l], B, room);
    P->i[l] = gemm_plan(B, L.in[l], L.out[l], room);
    P->off_w[l] = 0;
  }
  P->off_sums = P->off_rest = 0;
  const u64 first = (u64)L.in[0] * L.out[0];  // a split product's partial sums always fit; the sums of all columns have to
  P->first_kept = P->w[0].n_split > 1 && P->i[0].n_split == 1 && COLSUM_SLICES * cols <= first;
}

// The input as the products read it: fp32 is rounded to bf16 into the workspace, bf16 is read where it stands.  The products'
// loads to LDS take 16 bytes at a multiple of 16: an input that begins elsewhere goes to the workspace as well.
const bf16_t* tower_input(const MlpLayout& L, const float* d_pooled, const bf16_t* d_pooled_bf16, u32 B, char* ws, const WsLayout& S,
                          hipStream_t st) {
  const u64 n = (u64)B * L.in[0];
  bf16_t* h0 = (bf16_t*)(ws + S.off_h0);
  if (!d_pooled_bf16) {
    hipLaunchKernelGGL(k_cast_bf16, dim3(blocks_for(n / 4)), dim3(BLOCK), 0, st, d_pooled, h0, n);
    return h0;
  }
  const uintptr_t at = (uintptr_t)d_pooled_bf16;
  if (at % 16 == 0) return d_pooled_bf16;
  if (at % 8 == 0)
    hipLaunchKernelGGL(k_copy<uint2>, dim3(blocks_for(n / 4)), dim3(BLOCK), 0, st, (const uint2*)d_pooled_bf16, (uint2*)h0, n / 4);
  else
    hipLaunchKernelGGL(k_copy<bf16_t>, dim3(blocks_for(n)), dim3(BLOCK), 0, st, d_pooled_bf16, h0, n);
  return h0;
}

// Forward through the hidden layers; activations stay in the workspace.
bool forward_hidden(ctr_mlp* t, u32 replica, const bf16_t* h, u32 B, char* ws, const WsLayout& S, hipStream_t st) {
  const MlpLayout& L = t->L;
  const float* P = t->params + (u64)replica * t->M.stride;
  const bf16_t* PB = t->pb + (u64)replica * t->M.stride;
  for (u32 l = 0; l + 1 < L.n_layers; ++l) {
    bf16_t* a = (bf16_t*)(ws + S.off_act[l]);
    if (!product_forward(L, l, B, h, PB + L.w_off[l], P + L.w_off[l] + (u64)L.in[l] * L.out[l], a, ws, S, st)) return false;
    h = a;
  }
  return true;
}

}  // namespace

extern "C" {

size_t ctr_mlp_n_params(const ctr_mlp_config* cfg) {
  if (!mlp_config_ok(cfg)) return 0;
  MlpLayout L;
  make_layout(cfg, &L);
  return (size_t)L.n_params;
}

size_t ctr_mlp_bytes(const ctr_mlp_config* cfg) {
  if (!mlp_config_ok(cfg)) return 0;
  MlpLayout L;
  MemLayout M;
  make_layout(cfg, &L);
  mem_layout(cfg, L, &M);
  return M.total;
}

size_t ctr_mlp_workspace_bytes(const ctr_mlp_config* cfg, uint32_t batch) {
  if (!mlp_config_ok(cfg) || batch == 0 || batch % 8 != 0 || batch > CTR_MLP_MAX_BATCH) return 0;
  MlpLayout L;
  WsLayout S;
  make_layout(cfg, &L);
  ws_layout(cfg, L, batch, &S);
  return S.total;
}

int ctr_mlp_create(const ctr_mlp_config* cfg, void* d_mem, size_t bytes, void* hip_stream, ctr_mlp** out) {
  if (!cfg || !d_mem || !out) return CTR_E_INVAL;
  if (!mlp_config_ok(cfg)) return CTR_E_INVAL;
  if (((uintptr_t)d_mem & 255) != 0) return CTR_E_INVAL;
  ctr_mlp* t = new (std::nothrow) ctr_mlp();
  if (!t) return CTR_E_NOMEM;
  t->cfg = *cfg;
  make_layout(cfg, &t->L);
  mem_layout(cfg, t->L, &t->M);
  if (bytes < t->M.total) {
    delete t;
    return CTR_E_NOMEM;
  }
  t->mem = (char*)d_mem;
  t->params = (float*)(t->mem + t->M.off_params);
  t->m = (float*)(t->mem + t->M.off_m);
  t->v = (float*)(t->mem + t->M.off_v);
  t->pb = (bf16_t*)(t->mem + t->M.off_pb);
  t->vhat = cfg->kstep ? (float*)(t->mem + t->M.off_vhat) : nullptr;
  t->pend_mask = 0;
  hipStream_t st = (hipStream_t)hip_stream;
  hipLaunchKernelGGL(k_mlp_init, dim3(blocks_for(t->L.n_params)), dim3(BLOCK), 0, st, t->L,
                     cfg->init_seed * 0x9E3779B97F4A7C15ull, cfg->eps, cfg->n_replicas, t->M.stride, t->params, t->m,
                     t->v, t->vhat, t->pb);
  if (launch_status() != CTR_OK) {
    delete t;
    return CTR_E_DEVICE;
  }
  *out = t;
  return CTR_OK;
}

int ctr_mlp_destroy(ctr_mlp* t) {
  if (!t) return CTR_E_INVAL;
  delete t;
  return CTR_OK;
}

static int mlp_forward_impl(ctr_mlp* t, uint32_t replica, const float* d_pooled, const bf16_t* d_pooled_bf16,
                            uint32_t batch, float* d_logits, void* d_workspace, size_t workspace_bytes,
                            void* hip_stream) {
  if (!t || (!d_pooled && !d_pooled_bf16) || !d_logits || !d_workspace) return CTR_E_INVAL;
  if (replica >= t->cfg.n_replicas || batch == 0 || batch % 8 != 0 || batch > CTR_MLP_MAX_BATCH) return CTR_E_INVAL;
  if (((uintptr_t)d_workspace & 255) != 0) return CTR_E_INVAL;
  WsLayout S;
  ws_layout(&t->cfg, t->L, batch, &S);
  if (workspace_bytes < S.total) return CTR_E_NOMEM;
  hipStream_t st = (hipStream_t)hip_stream;
  char* ws = (char*)d_workspace;
  const MlpLayout& L = t->L;
  if (!forward_hidden(t, replica, tower_input(L, d_pooled, d_pooled_bf16, batch, ws, S, st), batch, ws, S, st)) return CTR_E_DEVICE;
  const u32 lo = L.n_layers - 1;
  const u64 base = (u64)replica * t->M.stride + L.w_off[lo];
  hipLaunchKernelGGL(k_out_forward, dim3(blocks_for((u64)batch * WAVE)), dim3(BLOCK), 0, st,
                     (const bf16_t*)(ws + S.off_act[lo - 1]), t->pb + base, t->params + base + L.in[lo], batch, L.in[lo],
                     d_logits);
  return launch_status();
}

// The gradient of the pooled input goes to d_grad_pooled (fp32) or to d_grad_pooled_bf16: exactly one is given.
static int mlp_step_impl(ctr_mlp* t, uint32_t replica, const float* d_pooled, const bf16_t* d_pooled_bf16,
                         const float* d_labels, uint32_t batch, float* d_grad_pooled, bf16_t* d_grad_pooled_bf16,
                         float* d_loss, void* d_workspace, size_t workspace_bytes, uint32_t mode, void* hip_stream) {
  if (!t || (!d_pooled && !d_pooled_bf16) || !d_labels || (!d_grad_pooled == !d_grad_pooled_bf16) || !d_loss ||
      !d_workspace)
    return CTR_E_INVAL;
  if (replica >= t->cfg.n_replicas || batch == 0 || batch % 8 != 0 || batch > CTR_MLP_MAX_BATCH) return CTR_E_INVAL;
  if (mode != CTR_STEP_LOCAL && mode != CTR_STEP_MERGE_PENDING) return CTR_E_INVAL;
  if (!t->cfg.kstep && mode != CTR_STEP_LOCAL) return CTR_E_INVAL;
  if (((uintptr_t)d_workspace & 255) != 0) return CTR_E_INVAL;
  WsLayout S;
  ws_layout(&t->cfg, t->L, batch, &S);
  if (workspace_bytes < S.total) return CTR_E_NOMEM;
  hipStream_t st = (hipStream_t)hip_stream;

  const MlpLayout& L = t->L;
  char* ws = (char*)d_workspace;
  const u32 B = batch;
  float* dlogit = (float*)(ws + S.off_dlogit);
  float* grads = (float*)(ws + S.off_grads);
  const float* P = t->params + (u64)replica * t->M.stride;
  const bf16_t* PB = t->pb + (u64)replica * t->M.stride;

  double* lterm = (double*)(ws + S.off_lterm);
  const bf16_t* h0 = tower_input(L, d_pooled, d_pooled_bf16, B, ws, S, st);
  if (!forward_hidden(t, replica, h0, B, ws, S, st)) return CTR_E_DEVICE;

  // output layer: logits, loss terms, and back through the last ReLU
  const u32 lo = L.n_layers - 1;
  const u32 Hl = L.in[lo];
  const bf16_t* a_last = (const bf16_t*)(ws + S.off_act[lo - 1]);
  bf16_t* dz_last = (bf16_t*)(ws + S.off_dz);
  const bf16_t* dz = dz_last;
  hipLaunchKernelGGL(k_out_step, dim3(blocks_for((u64)B * WAVE)), dim3(BLOCK), 0, st, a_last, PB + L.w_off[lo],
                     P + L.w_off[lo] + Hl, d_labels, B, Hl, dlogit, lterm, dz_last);

  const size_t n0 = (size_t)B * L.in[0];
  const bool in_place = d_grad_pooled ? overlap(h0, n0 * sizeof(bf16_t), d_grad_pooled, n0 * sizeof(float))
                                      : overlap(h0, n0 * sizeof(bf16_t), d_grad_pooled_bf16, n0 * sizeof(bf16_t));
  BackwardPlan plan;
  backward_plan(L, B, S.gemm_bytes, in_place, &plan);
  char* scratch = ws + S.off_gemm;
  GradSource src{};
  src.n_layers = L.n_layers;
  BatchSums q{};  // of all layers; taken behind the last product
  q.rows = B;
  q.partial = plan.first_kept ? grads + L.w_off[0] : (float*)(scratch + plan.off_sums);
  q.lterm = lterm;
  q.dlogit = dlogit;
  q.loss = d_loss;
  q.out_bias_grad = grads + L.w_off[lo] + Hl;
  u32 job_layer[COLSUM_MAX_JOBS];
  const auto add_sum = [&](u32 l, const bf16_t* x, const float* weight, u32 H, float* out) {
    const u32 j = q.n_jobs++;
    job_layer[j] = l;
    q.x[j] = x;
    q.weight[j] = weight;
    q.out[j] = out;
    q.H[j] = H;
    q.col0[j] = q.n_cols;
    q.n_cols += H;
    q.n_tiles += (H + COLSUM_TILE - 1) / COLSUM_TILE;
  };
  add_sum(lo, a_last, dlogit, Hl, grads + L.w_off[lo]);
  bool sums_taken = false;
  // hidden layers, last to first
  for (int l = (int)lo - 1; l >= 0; --l) {
    const bf16_t* h_prev = l == 0 ? h0 : (const bf16_t*)(ws + S.off_act[l - 1]);
    float* dw = grads + L.w_off[l];
    const GemmArgs w = weight_grad_args(L, (u32)l, B, h_prev, dz, dw);
    float* w_partial = (float*)(scratch + plan.off_w[l]);
    add_sum((u32)l, dz, nullptr, L.out[l], dw + (u64)L.in[l] * L.out[l]);
    // dH_prev[B x i] = dZ[B x o] W^T[o x i]: for the first layer the gradient of the pooled input; for a hidden
    // layer gated by the ReLU below and rounded to bf16 on the way out (the next dZ).  In a launch of its own it takes
    // the place of the activation that gates it, which nothing reads any more: an element is read and written by the
    // same thread.
    const bf16_t* mask = l == 0 ? nullptr : h_prev;
    bf16_t* below = l == 0 ? d_grad_pooled_bf16 : plan.paired[l] ? (bf16_t*)(scratch + plan.off_dz[l]) : (bf16_t*)(ws + S.off_act[l - 1]);
    const GemmArgs i = input_grad_args(L, (u32)l, B, dz, PB + L.w_off[l], l == 0 ? d_grad_pooled : nullptr, below, mask);
    if (plan.paired[l]) {
      if (!gemm_args_ok(false, false, w) || !gemm_args_ok(true, true, i)) return CTR_E_DEVICE;
      GemmArgs gw = w, gi = i;
      gemm_set_plan(gw, plan.w[l], w_partial);
      gemm_set_plan(gi, plan.i[l], nullptr);
      const u32 n_w = gw.tiles_m * gw.tiles_n * gw.n_split, n_i = gi.tiles_m * gi.tiles_n;
      sums_taken = l == 0;
      hipLaunchKernelGGL(k_gemm_backward, dim3(n_w + n_i + (l == 0 ? batch_sums_blocks(q) : 0)), dim3(BLOCK), 0, st, gw.A,
                         gw.B, gw, gi.A, gi.B, gi, n_w, n_i, q);
    } else {
      if (!gemm_args_ok(false, false, w) || !gemm_args_ok(true, true, i)) return CTR_E_DEVICE;
      const bool keep = plan.kept || (l == 0 && plan.first_kept);
      if (gemm_launch(false, false, w, plan.w[l], w_partial, keep, st) != hipSuccess) return CTR_E_DEVICE;
      if (gemm_launch(true, true, i, plan.i[l], (float*)(scratch + plan.off_rest), false, st) != hipSuccess) return CTR_E_DEVICE;
    }
    const bool split = (plan.kept || (l == 0 && plan.first_kept)) && plan.w[l].n_split > 1;
    src.weights[l] = {split ? w_partial : dw, (u64)L.in[l] * L.out[l], split ? plan.w[l].n_split : 1u};
    dz = below;
  }
  const bool sums_kept = plan.kept || plan.first_kept;
  if (sums_kept) {
    if (!sums_taken) hipLaunchKernelGGL(k_batch_sums, dim3(batch_sums_blocks(q)), dim3(BLOCK), 0, st, q);
  } else {
    // one pair of launches, unless the scratch ends before the columns do (layers of tens of thousands; each pair
    // writes the loss and the output bias's gradient, the same values every time)
    const BatchSums all = q;
    q.n_jobs = q.n_cols = q.n_tiles = 0;
    for (u32 j = 0; j < all.n_jobs; ++j) {
      add_sum(job_layer[j], all.x[j], all.weight[j], all.H[j], all.out[j]);
      const u64 next = j + 1 < all.n_jobs ? (u64)q.n_cols + all.H[j + 1] : ~0ull;
      if (next <= S.gemm_bytes / (COLSUM_SLICES * sizeof(float))) continue;
      hipLaunchKernelGGL(k_batch_sums, dim3(batch_sums_blocks(q)), dim3(BLOCK), 0, st, q);
      hipLaunchKernelGGL(k_batch_sums_final, dim3(blocks_for(q.n_cols)), dim3(BLOCK), 0, st, q);
      q.n_jobs = q.n_cols = q.n_tiles = 0;
    }
  }
  // dense optimizer
  for (u32 l = 0; l < L.n_layers; ++l) {
    src.w_off[l] = L.w_off[l];
    src.n_weights[l] = (u64)L.in[l] * L.out[l];
    src.biases[l] = {grads + L.w_off[l] + src.n_weights[l], 0, 1};
  }
  src.w_off[L.n_layers] = L.n_params;
  src.weights[lo] = {grads + L.w_off[lo], 0, 1};
  if (sums_kept)
    for (u32 j = 0; j < q.n_jobs; ++j)  // the first sum is the output layer's weight gradient, the others are of biases
      (j == 0 ? src.weights : src.biases)[job_layer[j]] = {q.partial + q.col0[j], q.n_cols, COLSUM_SLICES};
  const u32 amode = mode == CTR_STEP_MERGE_PENDING ? 2u : (t->cfg.kstep ? 1u : 0u);
  const u64 n4 = L.n_params >= DENSE_ADAM_WIDE_MIN ? L.n_params / 4 : 0;
  const DenseAdam adam = {(double)t->cfg.beta1, (double)t->cfg.beta2, (double)t->cfg.lr, amode};
  hipLaunchKernelGGL(k_dense_adam, dim3(blocks_for(L.n_params - 3 * n4)), dim3(BLOCK), 0, st,
                     t->params + (u64)replica * t->M.stride, t->m + (u64)replica * t->M.stride,
                     t->v + (u64)replica * t->M.stride, t->vhat, src, t->pb + (u64)replica * t->M.stride,
                     L.n_params, n4, adam);
  if (mode == CTR_STEP_MERGE_PENDING) t->pend_mask |= 1u << replica;
  return launch_status();
}

int ctr_mlp_forward(ctr_mlp* t, uint32_t replica, const float* d_pooled, uint32_t batch, float* d_logits,
                    void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (!d_pooled) return CTR_E_INVAL;
  return mlp_forward_impl(t, replica, d_pooled, nullptr, batch, d_logits, d_workspace, workspace_bytes, hip_stream);
}

int ctr_mlp_forward_bf16(ctr_mlp* t, uint32_t replica, const uint16_t* d_pooled_bf16, uint32_t batch,
                         float* d_logits, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (!d_pooled_bf16) return CTR_E_INVAL;
  return mlp_forward_impl(t, replica, nullptr, d_pooled_bf16, batch, d_logits, d_workspace, workspace_bytes,
                          hip_stream);
}

int ctr_mlp_step(ctr_mlp* t, uint32_t replica, const float* d_pooled, const float* d_labels, uint32_t batch,
                 float* d_grad_pooled, float* d_loss, void* d_workspace, size_t workspace_bytes, uint32_t mode,
                 void* hip_stream) {
  if (!d_pooled) return CTR_E_INVAL;
  return mlp_step_impl(t, replica, d_pooled, nullptr, d_labels, batch, d_grad_pooled, nullptr, d_loss, d_workspace,
                       workspace_bytes, mode, hip_stream);
}

int ctr_mlp_step_bf16(ctr_mlp* t, uint32_t replica, const uint16_t* d_pooled_bf16, const float* d_labels,
                      uint32_t batch, float* d_grad_pooled, float* d_loss, void* d_workspace,
                      size_t workspace_bytes, uint32_t mode, void* hip_stream) {
  if (!d_pooled_bf16) return CTR_E_INVAL;
  return mlp_step_impl(t, replica, nullptr, d_pooled_bf16, d_labels, batch, d_grad_pooled, nullptr, d_loss,
                       d_workspace, workspace_bytes, mode, hip_stream);
}

int ctr_mlp_step_bf16_grad_bf16(ctr_mlp* t, uint32_t replica, const uint16_t* d_pooled_bf16, const float* d_labels,
                                uint32_t batch, uint16_t* d_grad_pooled_bf16, float* d_loss, void* d_workspace,
                                size_t workspace_bytes, uint32_t mode, void* hip_stream) {
  if (!d_pooled_bf16 || !d_grad_pooled_bf16) return CTR_E_INVAL;
  return mlp_step_impl(t, replica, nullptr, d_pooled_bf16, d_labels, batch, nullptr, d_grad_pooled_bf16, d_loss,
                       d_workspace, workspace_bytes, mode, hip_stream);
}

// The tower's matrix product on its own (testing and measurement): C32[M x N] = A B.  tile = 0: as the tower runs it.
int ctr_debug_mlp_gemm(int a_k_contiguous, int b_k_contiguous, const uint16_t* d_a, uint32_t lda, const uint16_t* d_b,
                       uint32_t ldb, uint32_t m, uint32_t n, uint32_t k, float* d_c, uint32_t ldc, void* d_scratch,
                       size_t scratch_bytes, uint32_t tile, int split, void* hip_stream) {
  if (!d_a || !d_b || !d_c) return CTR_E_INVAL;
  if (m == 0 || n == 0 || k == 0 || ((m | n | k | lda | ldb | ldc) % 8u) != 0u) return CTR_E_INVAL;
  if (lda < (a_k_contiguous ? k : m) || ldb < (b_k_contiguous ? k : n) || ldc < n) return CTR_E_INVAL;
  if ((((uintptr_t)d_a | (uintptr_t)d_b | (uintptr_t)d_c | (uintptr_t)d_scratch) & 15) != 0) return CTR_E_INVAL;
  GemmArgs g{};
  g.A = d_a; g.lda = lda;
  g.B = d_b; g.ldb = ldb;
  g.M = m; g.N = n; g.K = k;
  g.C32 = d_c; g.ldc = ldc;
  g.epilogue = EPI_F32;
  const size_t room = d_scratch ? scratch_bytes : 0;
  if (!gemm_args_ok(a_k_contiguous != 0, b_k_contiguous != 0, g)) return CTR_E_INVAL;
  GemmPlan p;
  if (tile == 0)
    p = gemm_plan(m, n, k, room);
  else if (!gemm_plan_forced(m, n, k, room, tile, split != 0, &p))
    return CTR_E_INVAL;
  const hipError_t rc = gemm_launch(a_k_contiguous != 0, b_k_contiguous != 0, g, p, (float*)d_scratch, false, (hipStream_t)hip_stream);
  return rc == hipSuccess ? CTR_OK : CTR_E_DEVICE;
}

int ctr_mlp_gemm(int a_k_contiguous, int b_k_contiguous, const uint16_t* d_a, uint32_t lda, const uint16_t* d_b,
                 uint32_t ldb, uint32_t m, uint32_t n, uint32_t k, float* d_c, uint32_t ldc, void* d_scratch,
                 size_t scratch_bytes, void* hip_stream) {
  return ctr_debug_mlp_gemm(a_k_contiguous, b_k_contiguous, d_a, lda, d_b, ldb, m, n, k, d_c, ldc, d_scratch,
                            scratch_bytes, 0, 0, hip_stream);
}

int ctr_debug_mlp_gemm_plan(uint32_t m, uint32_t n, uint32_t k, size_t scratch_bytes, uint32_t* tile, uint32_t* items_per_tile,
                            uint32_t* ranges, uint32_t* range_length) {
  if (m == 0 || n == 0 || k == 0 || ((m | n | k) % 8u) != 0u || !tile || !items_per_tile || !ranges || !range_length)
    return CTR_E_INVAL;
  const GemmPlan p = gemm_plan(m, n, k, scratch_bytes);
  *tile = p.tile;
  *items_per_tile = p.n_split;
  *ranges = (k + p.k_per_sum - 1) / p.k_per_sum;
  *range_length = p.k_per_sum;
  return CTR_OK;
}

int ctr_debug_mlp_backward_plan(const ctr_mlp_config* cfg, uint32_t batch, int in_place, uint32_t* kept, uint32_t* paired,
                                uint32_t* weight_ranges, uint32_t* input_ranges) {
  if (!mlp_config_ok(cfg) || batch == 0 || batch % 8 != 0 || batch > CTR_MLP_MAX_BATCH) return CTR_E_INVAL;
  if (!kept || !paired || !weight_ranges || !input_ranges) return CTR_E_INVAL;
  MlpLayout L;
  make_layout(cfg, &L);
  BackwardPlan P;
  backward_plan(L, batch, gemm_scratch_bytes(cfg), in_place != 0, &P);
  *kept = P.kept ? 2u : P.first_kept ? 1u : 0u;
  for (u32 l = 0; l < cfg->n_hidden; ++l) {
    paired[l] = P.paired[l] ? 1u : 0u;
    weight_ranges[l] = P.w[l].n_split;
    input_ranges[l] = P.i[l].n_split;
  }
  return CTR_OK;
}

int ctr_mlp_kstep_merge(ctr_mlp* t, void* hip_stream) {
  if (!t || !t->cfg.kstep) return CTR_E_INVAL;
  hipStream_t st = (hipStream_t)hip_stream;
  hipLaunchKernelGGL(k_dense_merge, dim3(blocks_for(t->L.n_params)), dim3(BLOCK), 0, st, t->params, t->m, t->v,
                     t->vhat, t->pb, t->L.n_params, t->M.stride, t->cfg.n_replicas, t->pend_mask,
                     (double)t->cfg.lr);
  t->pend_mask = 0;
  return launch_status();
}

int ctr_mlp_export(ctr_mlp* t, uint32_t replica, float* h_params, float* h_m, float* h_v, float* h_vhat,
                   void* hip_stream) {
  if (!t || replica >= t->cfg.n_replicas) return CTR_E_INVAL;
  if (h_vhat && !t->vhat) return CTR_E_INVAL;
  hipStream_t st = (hipStream_t)hip_stream;
  const size_t nb = (size_t)t->L.n_params * sizeof(float);
  const u64 off = (u64)replica * t->M.stride;
  bool ok = true;
  if (h_params) ok = ok && hipMemcpyAsync(h_params, t->params + off, nb, hipMemcpyDeviceToHost, st) == hipSuccess;
  if (h_m) ok = ok && hipMemcpyAsync(h_m, t->m + off, nb, hipMemcpyDeviceToHost, st) == hipSuccess;
  if (h_v) ok = ok && hipMemcpyAsync(h_v, t->v + off, nb, hipMemcpyDeviceToHost, st) == hipSuccess;
  if (h_vhat) ok = ok && hipMemcpyAsync(h_vhat, t->vhat, nb, hipMemcpyDeviceToHost, st) == hipSuccess;
  ok = ok && hipStreamSynchronize(st) == hipSuccess;
  return ok ? CTR_OK : CTR_E_DEVICE;
}

int ctr_mlp_import(ctr_mlp* t, uint32_t replica, const float* h_params, const float* h_m, const float* h_v,
                   const float* h_vhat, uint32_t pending, void* hip_stream) {
  if (!t || replica >= t->cfg.n_replicas) return CTR_E_INVAL;
  if (h_vhat && !t->vhat) return CTR_E_INVAL;
  if (pending > 1 || (pending && !t->cfg.kstep)) return CTR_E_INVAL;
  hipStream_t st = (hipStream_t)hip_stream;
  const size_t nb = (size_t)t->L.n_params * sizeof(float);
  const u64 off = (u64)replica * t->M.stride;
  bool ok = true;
  if (h_params) ok = ok && hipMemcpyAsync(t->params + off, h_params, nb, hipMemcpyHostToDevice, st) == hipSuccess;
  if (h_m) ok = ok && hipMemcpyAsync(t->m + off, h_m, nb, hipMemcpyHostToDevice, st) == hipSuccess;
  if (h_v) ok = ok && hipMemcpyAsync(t->v + off, h_v, nb, hipMemcpyHostToDevice, st) == hipSuccess;
  if (h_vhat) ok = ok && hipMemcpyAsync(t->vhat, h_vhat, nb, hipMemcpyHostToDevice, st) == hipSuccess;
  if (!ok) return CTR_E_DEVICE;
  if (h_params)
    hipLaunchKernelGGL(k_refresh_bf16, dim3(blocks_for(t->L.n_params)), dim3(BLOCK), 0, st, t->params + off,
                       t->pb + off, t->L.n_params);
  ok = hipStreamSynchronize(st) == hipSuccess;  // the host arrays may be pageable: they are free again on return
  t->pend_mask = pending ? (t->pend_mask | (1u << replica)) : (t->pend_mask & ~(1u << replica));
  return ok ? launch_status() : CTR_E_DEVICE;
}

}  // extern "C"
