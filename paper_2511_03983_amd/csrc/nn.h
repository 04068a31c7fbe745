// Kernel launchers of the subnet training path (internal).  `bf16` selects the activation / weight
// storage type: 0 = fp32, 1 = bf16.  Residual stream, statistics, gradients of parameters: always fp32.
#pragma once
#include "twist_internal.h"

struct GemmEpilogue {
  float alpha = 1.f;             // out = alpha * (A.B + bias) + residual
  const void *bias = nullptr;    // [N], activation type
  const float *residual = nullptr;  // [M,N] fp32
  void *out = nullptr;           // [M,N]
  int out_f32 = 0;               // 1: out is fp32, 0: out is the activation type
  // Optional scratch for products with few output tiles and a long contraction (weight gradients): when given (and no
  // bias/residual is asked for) the contraction may be cut into parts whose fp32 partial products go here and are then
  // summed in a fixed order.
  float *splitk_ws = nullptr;
  size_t splitk_floats = 0;
  // Ungated activation of the output, as twist_act_fwd forms it from the stored one: act_out = f(out).  GEMM_NT with ldc = N on the context's stream and an
  // output of the model's type; anything else is refused.  With act_only the output itself need not be written (out is then scratch).
  void *act_out = nullptr;
  int act = 0;
  bool act_only = false;
  // Evaluation of a vocabulary projection: with `targets` the kernels of 256-row tiles may reduce each row of the (rounded) output to what its cross-entropy
  // needs instead of writing it: loss_parts[row][*loss_blocks][2] = (maximum, sum of exponentials against it) of a block of columns, and
  // target_logit[row].  *loss_blocks stays 0 where the output was written as usual; loss_parts may share its memory.
  const int32_t *targets = nullptr;
  float *loss_parts = nullptr, *target_logit = nullptr;
  int *loss_blocks = nullptr;
};
constexpr size_t kSplitkFloats = (size_t)256 * 256 * 256;

enum GemmLayout {
  GEMM_NT = 0,  // A [M,K] row-major, B [N,K] row-major         (y = x W^T)
  GEMM_NN = 1,  // A [M,K] row-major, B [K,N] row-major         (dx = dy W)
  GEMM_TN = 2   // A stored [K,M] row-major, B stored [K,N]     (dW = dy^T x)
};

// C[M,N] = epilogue( op(A) op(B) ), fp32 accumulation.  lda/ldb are the row strides of the stored operands.
// `st`: stream to enqueue on (null: the context's stream).
twist_status twist_gemm(twist_ctx *ctx, int bf16, GemmLayout lay, int M, int N, int K, const void *A, int64_t lda, const void *B,
                        int64_t ldb, int64_t ldc, const GemmEpilogue &ep, hipStream_t st = nullptr);

// Weight gradients over the same K rows, up to kGroupProducts of them: one launch where their kernels allow it.  `scratch` (or null) as in
// GemmEpilogue; chosen as in twist_weight_grads_raw.
using WeightGrad = twist_weight_grad;
constexpr int kGroupProducts = 4;
twist_status twist_weight_grads(twist_ctx *ctx, int bf16, int n, const WeightGrad *items, int K, float *scratch, size_t scratch_floats, hipStream_t st = nullptr,
                                int32_t *chosen = nullptr);

// What the rule that chooses bf16 kernels expects (host only), added up: microseconds, and those that CUs without a tile stand idle.  Several
// M, N: weight gradients in one launch.
struct GemmEstimate { double us = 0.0, idle = 0.0; };
void twist_gemm_estimate(GemmLayout lay, int n, const int *Ms, const int *Ns, int K, bool f32_out, size_t split_floats, GemmEstimate &sum);

// the bf16 ping-pong kernel for GEMM_NT (ep: a gemm_tile.h Ep), tiles of 256 x bn, bn = 256 or 128; with `targets` the rows' loss parts instead of an output
void twist_launch_gemm_nt(hipStream_t st, int bn, int M, int N, int K, const uint16_t *a, int64_t lda, const uint16_t *b, int64_t ldb, const void *ep,
                          const int32_t *targets = nullptr, float *loss_parts = nullptr, float *target_logit = nullptr);
// the bf16 kernels for tiles of 64 and 32 (ep: a gemm_tile.h Ep), the contraction cut into `parts` parts of kchunk (a multiple of 128)
void twist_launch_gemm_dl(hipStream_t st, int tile, GemmLayout lay, int M, int N, int K, const uint16_t *a, int64_t lda, const uint16_t *b, int64_t ldb, const void *ep,
                          int parts, int kchunk);
// the same for the weight gradients of a group (a gemm_tile.h TnGroup), `tiles` in all
void twist_launch_gemm_dl_group(hipStream_t st, int tile, const void *group, int tiles, int K, const void *ep, int parts, int kchunk);
// the bf16 kernels whose two groups of waves share the contraction: tiles of 128x192, 192x128, 128x128, 128x96 and 64x96; otherwise as the two above
void twist_launch_gemm_kp(hipStream_t st, int bm, int bn, GemmLayout lay, int M, int N, int K, const uint16_t *a, int64_t lda, const uint16_t *b, int64_t ldb,
                          const void *ep, int parts, int kchunk);
void twist_launch_gemm_kp_group(hipStream_t st, int bm, int bn, const void *group, int tiles, int K, const void *ep, int parts, int kchunk);
// the fp32 form of twist_gemm, and the sum of the partial products [parts][M][N] of a product whose contraction was cut
// (out = alpha * sum in ascending order)
twist_status twist_gemm_f32(twist_ctx *ctx, hipStream_t st, GemmLayout lay, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb,
                            int64_t ldc, const GemmEpilogue &e);
// its tile, number of parts of the contraction and length of a part (vec: bases and strides allow 16-byte loads)
void twist_gemm_f32_choice(const twist_ctx *ctx, GemmLayout lay, int M, int N, int K, bool vec, bool may_split, size_t split_floats, int &tile, int &parts, int &kchunk);
// weight gradients in fp32 that share a launch (aligned operands; `first`: number of a product's first tile; out: part 0 of a cut contraction): the choice
// as above (false: none that sums as finely as separate launches), and the launch
struct F32Product {
  const float *a, *b;
  float *out;
  int64_t lda, ldb;
  int M, N, first, tiles_m, tiles_n;
  float alpha;
};
bool twist_gemm_f32_group_choice(int n, const int *Ms, const int *Ns, int K, size_t split_floats, int &tile, int &parts, int &kchunk);
void twist_launch_gemm_f32_group(hipStream_t st, int tile, int n, const F32Product *products, int tiles, int K, int parts, int kchunk);
twist_status twist_splitk_reduce(twist_ctx *ctx, hipStream_t st, const float *parts_ws, int parts, int M, int N, void *out, int64_t ldc, int out_f32,
                                 float alpha);

// causal multi-head attention on a fused qkv buffer [T, 3*Hs*dh] (q | k | v); o [T, Hs*dh]; lse [B,Hs,N] fp32.
// o32 (may be null): the same output unrounded, [T, Hs*dh] fp32, written for bf16 models by every tiled kernel (in bf16 and in fp32
// arithmetic), not by the plain ones; the tiled backward kernels need it (without it, or on shapes they do not cover, the plain kernels run).
// keep (may be null; device, one entry per head): heads with keep[h] < 0 are masked (Masked TwIST, Section 4.1): the forward
// kernels write zeros for them, the backward kernels zero gradients, and neither visits their keys.
twist_status twist_attention_fwd(twist_ctx *ctx, int bf16, const void *qkv, void *o, float *o32, float *lse, int B, int N, int Hs, int dh,
                                 const int32_t *keep = nullptr);
// dqkv [T, 3*Hs*dh] from do [T, Hs*dh]; delta [B,Hs,N] fp32 scratch (sum_j p_ij dp_ij, written by the dq pass).
// o_f32: the forward output in fp32 (bf16 models: the unrounded copy o32; fp32 models: o itself; null: the plain kernels run).
// rope_tab (may be null): the table of twist_rope_table; when given, the q and k gradients are also taken back through
// the rotary embedding (inside the tiled kernels where they cover the shape, else by twist_rope_apply afterwards).
twist_status twist_attention_bwd(twist_ctx *ctx, int bf16, const void *qkv, const float *o_f32, const void *dout, const float *lse, float *delta,
                                 void *dqkv, int B, int N, int Hs, int dh, const float *rope_tab, const int32_t *keep = nullptr);
// bf16 models outside flash.hip's tiles: the kernels with fp32 probabilities on the bf16 instruction, and whether they cover the operands
// (null: not asked about)
bool twist_attention_64_ok(const twist_ctx *ctx, const void *qkv, const void *o, const void *o32, const void *dout, const void *dqkv, int N, int Hs, int dh);
twist_status twist_attention_64_fwd(twist_ctx *ctx, const void *qkv, void *o, float *o32, float *lse, int B, int N, int Hs, int dh, const int32_t *keep,
                                    bool rounded);
twist_status twist_attention_64_bwd(twist_ctx *ctx, const void *qkv, const float *o32, const void *dout, const float *lse, float *delta, void *dqkv, int B, int N, int Hs, int dh,
                                    const float *rope_tab, const int32_t *keep, bool rounded, bool *rope_done);
// the tiled fp32 kernels behind the two calls above, and whether they cover the operands
bool twist_attention_f32_ok(const twist_ctx *ctx, const void *qkv, const void *o, const void *dout, const void *dqkv, int dh);
twist_status twist_attention_f32_fwd(twist_ctx *ctx, int bf16, const void *qkv, void *o, float *o32, float *lse, int B, int N, int Hs, int dh, const int32_t *keep);
twist_status twist_attention_f32_bwd(twist_ctx *ctx, int bf16, const void *qkv, const float *o, const void *dout, const float *lse, float *delta, void *dqkv, int B, int N,
                                     int Hs, int dh, const int32_t *keep);

twist_status twist_embed_fwd(twist_ctx *ctx, int bf16, const int32_t *tok, const void *tok_embed, const void *pos_embed, float *x, int B, int N, int D, int vocab);
twist_status twist_embed_bwd(twist_ctx *ctx, const int32_t *tok, const float *dx, float *d_tok, float *d_pos, int B, int N, int D);
twist_status twist_zero_f32(twist_ctx *ctx, float *p, int64_t n);
twist_status twist_cast_in(twist_ctx *ctx, int bf16, const void *src, float *dst, int64_t n);

// y = norm(x) * w (+ b); stats[2*T] = (mean or 0, rstd) per row
twist_status twist_norm_fwd(twist_ctx *ctx, int bf16, int rms, const float *x, const void *w, const void *b, void *y, float *stats, int T, int D, float eps);
// dx (+)= norm backward of dy; dxb = activation-type copy of the resulting dx (may be null);
// dw, db (fp32, overwritten; db may be null); partial: scratch of at least norm_partial_floats(T, D).
// With defer_reduce the per-chunk partial sums are left in `partial` and dw/db are not written: the caller later sums
// many such buffers with one twist_col_reduce_batch launch (items {partial, dw, 2 D, D, 1} and {partial + D, db, 2 D, D, 1};
// same summation order, hence the same bits).  csum (may be null): per-chunk column sums of dxb, as twist_colsum defers them.
twist_status twist_norm_bwd(twist_ctx *ctx, int bf16, int rms, const void *dy, const float *x, const void *w, const float *stats, float *dx,
                            int accumulate, void *dxb, float *dw, float *db, float *partial, int T, int D, bool defer_reduce = false,
                            float *csum = nullptr);
size_t twist_norm_partial_floats(int T, int D);
// One deferred column reduction: out[c] = alpha * sum over the T/16-row chunks k of partial[k * stride + c], c < n.
struct ColReduce {
  const float *partial;
  float *out;
  int64_t stride;
  int n;
  float alpha;
};
twist_status twist_col_reduce_batch(twist_ctx *ctx, const ColReduce *items, int n_items, int T);

// column sums: out[n] = alpha * sum_t src[t, n] (fp32, overwritten); partial scratch >= colsum_partial_floats.
// With defer_reduce only the per-chunk sums are written (stride Ncols); the caller reduces them later in a batch.
twist_status twist_colsum(twist_ctx *ctx, int bf16, const void *src, int64_t ld, float alpha, float *out, float *partial, int T, int Ncols,
                          bool defer_reduce = false);
size_t twist_colsum_partial_floats(int T, int Ncols);

// cos/sin table [N, dh/2, 2] (computed in fp64), then in-place rotation of the q and k heads of a fused qkv buffer
twist_status twist_rope_table(twist_ctx *ctx, float *tab, int N, int dh, float theta);
twist_status twist_rope_apply(twist_ctx *ctx, int bf16, void *qkv, const float *tab, int B, int N, int Hs, int dh, float sign);

// act: a = f(u) (gu = [T,F]) or a = silu(g) * u (gu = [T,2F], gate first).
// keep (may be null; device, one entry per FFN block of `unit` neurons): blocks with keep[b] < 0 are masked (Masked TwIST,
// Section 4.1): their activations are written as zero and, in the backward kernel, da is taken as zero there.
// sums (may be null): also the column sums of dgu per chunk of rows, twist_colsum_partial_floats(T, columns of dgu) of them.
twist_status twist_act_fwd(twist_ctx *ctx, int bf16, int act, const void *gu, void *a, int T, int F, const int32_t *keep = nullptr, int unit = 1);
twist_status twist_act_bwd(twist_ctx *ctx, int bf16, int act, const void *gu, const void *da, void *dgu, int T, int F, const int32_t *keep = nullptr,
                           int unit = 1, float *sums = nullptr);

// logits [T,V] -> in place dlogits = (softmax - onehot)/T (grad) or left alone; row losses to rowloss[T]; then loss = mean
twist_status twist_ce_fwd_bwd(twist_ctx *ctx, int bf16, void *logits, int64_t ld, const int32_t *targets, float *rowloss, float *loss, int T, int V, bool grad = true);
// the same loss from the parts that a projection left (GemmEpilogue::targets); rowloss holds the target logits and receives the row losses
twist_status twist_ce_parts(twist_ctx *ctx, const float *parts, int blocks, float *rowloss, float *loss, int T);
// dx = 2 (x - y)/n ; dxb = activation-type copy; loss = mean squared error
twist_status twist_mse_fwd_bwd(twist_ctx *ctx, int bf16, const float *x, const void *y, float *dx, void *dxb, float *partial, float *loss, int64_t n);

twist_status twist_sgd(twist_ctx *ctx, int bf16, void *params, float *master, const float *grads, int64_t n, float lr);
twist_status twist_adamw(twist_ctx *ctx, int bf16, void *params, float *master, const float *grads, float *m, float *v, int64_t n, int64_t n_decay,
                         float lr, float b1, float b2, float eps, float wd, int64_t step);
