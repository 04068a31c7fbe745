// One forward + backward pass of a dense subnet, and the local optimizer step ("True TwIST" worker,
// Section 4.1): pre-norm transformer layer of Appendix A.2 at the subnet's own width, module outputs
// scaled by sqrt(N_full / N_sub) before each residual add (Section 3.4).
//
// Host orchestration only: every step is a kernel from nn.hip / gemm.hip / attention.hip enqueued on the
// context's stream.  Activations needed by the backward pass are kept in the caller's workspace.
#include <cmath>

#include "nn.h"

namespace {

// Bump allocator over the workspace; with base == nullptr it only measures.
struct Carver {
  char *base;
  size_t off = 0;
  explicit Carver(void *b) : base(static_cast<char *>(b)) {}
  template <class T = void> T *take(size_t bytes) {
    off = align_up(off, 256);
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += bytes;
    return p;
  }
};

struct LayerBufs {
  void *h1, *qkv, *o, *h2, *gu, *a;
  float *lse, *o32;  // o32: unrounded attention output (bf16 models), feeds the backward pass's delta
};

// Masked TwIST on the kept blocks only: the kept blocks of a layer's partitioned tensors are gathered into a scratch copy of one
// layer, the layer runs dense at its kept width, and its gradients are spread back with zeros in the masked blocks.  The scratch
// holds one layer at a time (weights again for the backward pass), and the whole has to fit the workspace that the full-width pass is
// sized for: the activations of every layer shrink with the width, the scratch is that of one layer.  (Llama-1B widths, half the
// blocks: 150 MB of scratch against 54 KB per token and layer, i.e. 2800 tokens for one layer, 130 for 22.)
struct Compact {
  bool on = false;
  int64_t off[TWIST_N_LAYER_TENSORS];       // element offsets of one layer's matrices and (behind them) biases in the scratch
  int64_t elems = 0, bias_off = 0;          // all of them; where the biases start
};

struct Workspace {
  char *cw;                   // compact masked pass: weights of the layer at work,
  float *cg, *cb;             // its matrix gradients, and the partitioned bias gradients of all layers (elems - bias_off each)
  int64_t cb_stride;
  std::vector<float *> xs;    // residual stream before / inside / after every layer, fp32 [T,D]
  std::vector<float *> stats; // (mean, rstd) per row for each norm
  std::vector<LayerBufs> layer;
  float *dx, *rope_tab, *rowloss, *delta;
  float *splitk;        // scratch of the weight-gradient projections that are cut along the token dimension
  float *norm_partial;  // one block of per-chunk norm-gradient sums per norm layer (2 n_layers + 1), reduced in one launch at the end
  size_t norm_partial_stride;
  float *bias_partial;  // models with biases: per layer, the per-chunk column sums behind the four bias gradients
  size_t bias_partial_stride;
  void *dxb, *dxb2, *hf, *logits, *da, *dgu, *dh, *dout, *dqkv;
  int64_t ld_logits;
  size_t bytes;
};

// offsets of layer l's kept blocks in the scratch (tensors whose blocks are all kept are used where they are: -1)
void compact_layout(const twist_model_desc &d, const twist_plan *plan, int l, Compact &c) {
  static const int order[] = {TWIST_WQ, TWIST_WK, TWIST_WV, -1, TWIST_WO, -1, TWIST_W_GATE, TWIST_W_UP, -1, TWIST_W_DOWN, -2, TWIST_BQ, TWIST_BK, TWIST_BV, -1, TWIST_B_UP, -1};
  std::fill(c.off, c.off + TWIST_N_LAYER_TENSORS, (int64_t)-1);
  int64_t n = 0;
  for (int t : order) {
    if (t < 0) {
      n = (int64_t)align_up((size_t)n, 64);
      if (t == -2) c.bias_off = n;
      continue;
    }
    const PlanEntry &pe = plan->at(l, twist_tensor_kind(d, t));
    if (pe.n_sub == pe.n_full) continue;
    int r, cc;
    twist_tensor_shape(d, t, pe.n_sub, pe.n_sub, r, cc);
    if (!r) continue;
    c.off[t] = n;
    n += (int64_t)r * cc;
  }
  c.elems = n;
}

// heads / ffn: width of every layer in heads and FFN blocks; cplan: the plan whose row is compacted, or null
void carve(const twist_ctx *ctx, const std::vector<int32_t> &heads, const std::vector<int32_t> &ffn, const twist_plan *cplan, int B, int N, void *base, Workspace &w) {
  const twist_model_desc &d = ctx->d;
  const size_t es = ctx->esize();
  const size_t T = (size_t)B * N, D = d.d_model;
  const int nf = d.act == TWIST_ACT_SWIGLU ? 2 : 1;
  Carver c(base);
  w.xs.resize(2 * d.n_layers + 1);
  w.stats.resize(2 * d.n_layers + 1);
  for (auto &p : w.xs) p = c.take<float>(T * D * 4);
  for (auto &p : w.stats) p = c.take<float>(T * 2 * 4);
  w.layer.resize(d.n_layers);
  size_t hd_max = 0, f_max = 0, h_max = 0;
  for (int l = 0; l < d.n_layers; ++l) {
    const size_t HD = (size_t)heads[l] * d.d_head, F = (size_t)ffn[l] * d.ffn_granule;
    hd_max = std::max(hd_max, HD); f_max = std::max(f_max, F); h_max = std::max(h_max, (size_t)heads[l]);
    LayerBufs &b = w.layer[l];
    b.h1 = c.take(T * D * es);
    b.qkv = c.take(T * 3 * HD * es);
    b.o = c.take(T * HD * es);
    b.o32 = es == 2 ? c.take<float>(T * HD * 4) : nullptr;
    b.lse = c.take<float>((size_t)B * heads[l] * N * 4);
    b.h2 = c.take(T * D * es);
    b.gu = c.take(T * nf * F * es);
    b.a = c.take(T * F * es);
  }
  w.dx = c.take<float>(T * D * 4);
  w.dxb = c.take(T * D * es);
  w.dxb2 = c.take(T * D * es);
  w.hf = c.take(T * D * es);
  w.ld_logits = (int64_t)align_up((size_t)d.vocab, 8);
  w.logits = d.vocab ? c.take(T * w.ld_logits * es) : nullptr;
  w.rowloss = c.take<float>(std::max<size_t>(T, 1024) * 4);
  w.rope_tab = c.take<float>((size_t)N * d.d_head * 4);
  w.splitk = c.take<float>(kSplitkFloats * 4);
  w.norm_partial_stride = align_up(twist_norm_partial_floats((int)T, (int)D), 64);
  w.norm_partial = c.take<float>(w.norm_partial_stride * (2 * (size_t)d.n_layers + 1) * 4);
  w.bias_partial_stride = d.has_bias ? align_up(twist_colsum_partial_floats((int)T, (int)(2 * D + nf * f_max + 3 * hd_max)), 64) : 0;
  w.bias_partial = c.take<float>(w.bias_partial_stride * (size_t)d.n_layers * 4);
  w.delta = c.take<float>((size_t)B * h_max * N * 4);
  w.da = c.take(T * f_max * es);
  w.dgu = c.take(T * nf * f_max * es);
  w.dh = c.take(T * D * es);
  w.dout = c.take(T * hd_max * es);
  w.dqkv = c.take(T * 3 * hd_max * es);
  if (cplan) {
    int64_t most = 0, bias = 0;
    for (int l = 0; l < d.n_layers; ++l) {
      Compact k;
      compact_layout(d, cplan, l, k);
      most = std::max(most, k.elems);
      bias = std::max(bias, k.elems - k.bias_off);
    }
    w.cw = c.take<char>((size_t)most * es);
    w.cg = c.take<float>((size_t)most * 4);
    w.cb_stride = (int64_t)align_up((size_t)bias, 64);
    w.cb = c.take<float>((size_t)w.cb_stride * d.n_layers * 4);
  }
  w.bytes = align_up(c.off, 256);
}

// The weight-gradient projections of the backward pass only write parameter gradients, and nothing downstream in the pass reads them.
// They are either enqueued on a second stream, where they run next to the chain of input-gradient kernels and fill the CUs that the
// chain leaves idle, each by itself or the FFN's two and the attention's two together; or in one launch at the layer's end.  Slot i
// (0 = FFN down, 1 = FFN up/gate or both, 2 = attention output, 3 = q/k/v or both) has a "ready" event (the main stream has produced
// the operands) and a "done" event (the side stream has consumed them; the main stream waits for it before it overwrites them).
struct Schedule {
  bool whole = true;  // a layer's gradients in one launch on the caller's stream; otherwise on the second stream, and:
  bool ffn_pair = false, attn_pair = false;
  // T tokens, `heads` columns of heads and F of the FFN's hidden layer in an average layer.
  // Where the gradients are few the events and waits, about 12 us of host time per layer and gaps of a few us each on the device, cost
  // more than the overlap gives.  Forward and backward of 6 layers, us, second stream / one stream:
  //   bf16 (apart), 0.05 GFLOP 974 / 596    0.8 983 / 744    3.2 1012 / 897    12.9 1338 / 1316   (pairs / one launch) 14.5 1490 / 1522    21 2013 / 2079
  //   fp32          0.9 GFLOP 1263 / 1048   1.1 1454 / 1222   2.1 1598 / 1433   3.2 1604 / 1571   6.4 2013 / 1991   7.2 2034 / 2083   14.5 2964 / 3097
  // The second stream's launches fill the CUs that the chain and they themselves leave idle, which one launch does not do; but it is the shorter one
  // for small layers, and has no events, waits and gaps (about 14 us a layer).  Estimates are of the kernels that run.  Of 126 bf16 models of 13 to 1900
  // GFLOP a layer the form taken is 0.4 % above the fastest on average, and 2 to 6 % for 11 of them.  d x tokens (columns of heads, hidden), us of a
  // pass of 6 layers, second stream / one launch: 768 x 2048 (384, 1536) 1390 / 1317, 576 x 6144 (128, 1152) 1846 / 1718, 768 x 8192 (768, 3072) 5110 / 4938,
  // 1024 x 1024 (1024, 1408 gated) 1587 / 1450; and on the other side of the line 896 x 6144 (512, 2464 gated) 3570 / 3709, 1536 x 2048 (384, 3072) 2270 / 2349,
  // 2560 x 4096 (2560, 5120) 10089 / 11071.
  void choose(bool bf16, int T, int D, int heads, int F, int nf) {
    const double flop = 2.0 * T * D * (4.0 * heads + (nf + 1.0) * F);
    whole = flop < (bf16 ? 13e9 : 3e9);
    if (!whole && bf16) {
      // a launch for two where it is expected to take a twentieth less than two launches: 1536 x 3000 (1536, 3072) 3830 a pass, apart 4029; not the FFN's
      // of 8192 x 2048 x 2816, whose 264 tiles would take two rounds: 10417, 9853.  (Without the twentieth 126 models take 0.2 % longer on average.)
      const int f = nf * F, q = 3 * heads, Ms[4] = {D, f, D, q}, Ns[4] = {F, D, heads, D};
      GemmEstimate chain, one[4], two[2], all;
      twist_gemm_estimate(GEMM_NN, 1, &T, &F, D, false, 0, chain);
      twist_gemm_estimate(GEMM_NN, 1, &T, &D, f, false, 0, chain);
      twist_gemm_estimate(GEMM_NN, 1, &T, &heads, D, false, 0, chain);
      twist_gemm_estimate(GEMM_NN, 1, &T, &D, q, false, 0, chain);
      for (int i = 0; i < 4; ++i) twist_gemm_estimate(GEMM_TN, 1, Ms + i, Ns + i, T, true, kSplitkFloats, one[i]);
      for (int i = 0; i < 2; ++i) twist_gemm_estimate(GEMM_TN, 2, Ms + 2 * i, Ns + 2 * i, T, true, kSplitkFloats, two[i]);
      twist_gemm_estimate(GEMM_TN, 4, Ms, Ns, T, true, kSplitkFloats, all);
      bool pair[2];
      GemmEstimate side = chain;  // the chain, and the launches of the second stream
      for (int i = 0; i < 2; ++i) {
        const GemmEstimate apart{one[2 * i].us + one[2 * i + 1].us, one[2 * i].idle + one[2 * i + 1].idle}, &less = two[i].us < apart.us ? two[i] : apart;
        pair[i] = two[i].us < 0.95 * apart.us;
        side.us += less.us;
        side.idle += less.idle;
      }
      ffn_pair = pair[0];
      attn_pair = pair[1];
      whole = chain.us + all.us + side.idle < side.us + 14.0;
    }
  }
};

struct SideStream : Schedule {
  twist_ctx *ctx;
  bool on = false, recorded[4] = {false, false, false, false};  // on the second stream (same launches, so the same results, without it)
  explicit SideStream(twist_ctx *c) : ctx(c) {}
  twist_status init(int T, int D, int heads, int F, int nf) {
    choose(ctx->d.dtype == TWIST_BF16, T, D, heads, F, nf);
    on = !whole && ctx->overlap;
    if (!on) return TWIST_OK;
    if (!ctx->side) {
      TW_HIP(ctx, hipStreamCreateWithFlags(&ctx->side, hipStreamNonBlocking));
      for (int i = 0; i < 4; ++i) {
        TW_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_ready[i], hipEventDisableTiming));
        TW_HIP(ctx, hipEventCreateWithFlags(&ctx->ev_done[i], hipEventDisableTiming));
      }
    }
    return TWIST_OK;
  }
  hipStream_t stream() const { return on ? ctx->side : nullptr; }
  twist_status fork(int i) {  // everything enqueued on the main stream so far precedes the side stream's next kernel
    if (!on) return TWIST_OK;
    TW_HIP(ctx, hipEventRecord(ctx->ev_ready[i], ctx->stream));
    TW_HIP(ctx, hipStreamWaitEvent(ctx->side, ctx->ev_ready[i], 0));
    return TWIST_OK;
  }
  twist_status done(int i) {
    if (!on) return TWIST_OK;
    TW_HIP(ctx, hipEventRecord(ctx->ev_done[i], ctx->side));
    recorded[i] = true;
    return TWIST_OK;
  }
  twist_status wait_done(int i) {  // the main stream may overwrite slot i's operands after this
    if (!on || !recorded[i]) return TWIST_OK;
    TW_HIP(ctx, hipStreamWaitEvent(ctx->stream, ctx->ev_done[i], 0));
    return TWIST_OK;
  }
};

twist_status check_train_shape(twist_ctx *ctx, const twist_subnet *sub, int B, int N) {
  const twist_model_desc &d = ctx->d;
  if (B < 1 || N < 1) TW_FAIL(ctx, TWIST_ESHAPE, "fwd_bwd: batch %d x %d tokens is empty", B, N);
  if (N > d.max_seq) TW_FAIL(ctx, TWIST_ESHAPE, "fwd_bwd: %d tokens exceed max_seq=%d", N, d.max_seq);
  if (d.has_bias && d.act == TWIST_ACT_SWIGLU) TW_FAIL(ctx, TWIST_ESHAPE, "fwd_bwd: gated FFN with biases is not supported");
  if (d.d_head > 256) TW_FAIL(ctx, TWIST_ESHAPE, "fwd_bwd: d_head=%d above 256 is not supported", d.d_head);
  if ((int64_t)B * N * std::max(d.d_model, d.vocab) >= (1ll << 40)) TW_FAIL(ctx, TWIST_ESHAPE, "fwd_bwd: batch too large");
  (void)sub;
  return TWIST_OK;
}

}  // namespace

twist_status twist_train_workspace_bytes(twist_ctx *ctx, const twist_subnet *sub, int B, int N, size_t *bytes) {
  TW_TRY(check_train_shape(ctx, sub, B, N));
  Workspace w;
  carve(ctx, sub->plan->layout.heads_sub, sub->plan->layout.ffn_sub, nullptr, B, N, nullptr, w);
  *bytes = w.bytes;
  return TWIST_OK;
}

// Whether the masked pass under a row of `plan` runs on the kept blocks only (struct Compact).  That depends on the model, the blueprint's
// widths and the batch alone, not on the buffers of one call: equal calls take the same form and give the same bits.
// Compacting moves about 12 r + 4 bytes per layer parameter (bf16, r = kept share: gathered twice, gradients spread once) at
// 4.5 TB/s and saves 6 T (1 - r) flop of it at about 0.9 PFLOP/s (fp32 models: 20 r + 4 bytes, 0.1 PFLOP/s), which is where the
// line lies.  Llama-1B widths, 6 layers, 4 x 2048 tokens, half the blocks: 13.9 ms against 20.4 in place.
// Kept widths that break the 16-byte rows of a width that has them lose the matrix-core kernels in bf16 (2 such layers with 2501 of
// 5632 neurons: 28.6 ms against 6.0 in place), so those models stay in place; in fp32 the projections go on with scalar loads, which
// costs them up to 0.4 of their time (4 layers of 768, 1533 of 3072 neurons, 2 x 512 tokens: 2.6 ms; 1536 neurons 2.0; in place 2.8).
bool twist_train_masked_compact(const twist_ctx *ctx, const twist_plan *plan, int B, int N) {
  const twist_model_desc &d = ctx->d;
  const int L = d.n_layers, T = B * N;
  const int vec = 16 / ctx->esize();
  double full_p = 0, kept_p = 0;
  bool odd = false;  // some kept width breaks 16-byte rows
  for (int l = 0; l < L; ++l) {
    if (!twist_expand_fits(ctx, plan, l)) return false;
    const int q[2] = {d.d_head, d.ffn_granule};
    for (int k = 0; k < 2; ++k) odd |= plan->at(l, k).n_full * q[k] % vec == 0 && plan->at(l, k).n_sub * q[k] % vec != 0;
    for (int t = TWIST_WQ; t <= TWIST_W_DOWN; ++t) {
      const PlanEntry &pe = plan->at(l, twist_tensor_kind(d, t));
      int r, c;
      twist_tensor_shape(d, t, d.n_heads, ctx->n_ffn_units(), r, c);
      full_p += (double)r * c;
      kept_p += (double)r * c * pe.n_sub / pe.n_full;
    }
  }
  if (odd && d.dtype == TWIST_BF16) return false;
  const double r = kept_p / full_p, gain = T * (1.0 - (odd ? 1.4 : 1.0) * r), cost = d.dtype == TWIST_BF16 ? 33.0 * (12.0 * r + 4.0) : 4.0 * (20.0 * r + 4.0);
  if (gain <= cost) return false;
  std::vector<int32_t> h1(L, d.n_heads), f1(L, ctx->n_ffn_units()), h2(L), f2(L);
  for (int l = 0; l < L; ++l) { h2[l] = plan->at(l, TWIST_KIND_HEAD).n_sub; f2[l] = plan->at(l, TWIST_KIND_FFN).n_sub; }
  Workspace full, kept;
  carve(ctx, h1, f1, nullptr, B, N, nullptr, full);
  carve(ctx, h2, f2, plan, B, N, nullptr, kept);
  return kept.bytes <= full.bytes;  // the caller's workspace is sized for the pass in place
}

twist_status twist_train_fwd_bwd(twist_ctx *ctx, twist_subnet *sub, const void *inputs, const void *targets, int B, int N, void *ws,
                                 size_t ws_bytes, float *loss_dev, bool forward_only, const twist_plan *mask_plan, int mask_row) {
  TW_TRY(check_train_shape(ctx, sub, B, N));
  if (!forward_only && !sub->grads) TW_FAIL(ctx, TWIST_ESHAPE, "fwd_bwd: subnet was extracted without gradient storage");
  if (reinterpret_cast<uintptr_t>(ws) % 256) TW_FAIL(ctx, TWIST_ESHAPE, "fwd_bwd: workspace must be 256-byte aligned");
  Workspace w;
  const SubLayout &L = sub->plan->layout;
  carve(ctx, L.heads_sub, L.ffn_sub, nullptr, B, N, ws, w);
  if (ws_bytes < w.bytes) TW_FAIL(ctx, TWIST_ESHAPE, "fwd_bwd: workspace of %zu bytes is smaller than the %zu needed", ws_bytes, w.bytes);

  const twist_model_desc &d = ctx->d;
  const int bf = d.dtype == TWIST_BF16, es = ctx->esize();
  const int T = B * N, D = d.d_model, dh = d.d_head;
  const int rms = d.norm == TWIST_NORM_RMS;
  const int nf = d.act == TWIST_ACT_SWIGLU ? 2 : 1;
  const bool lm = d.vocab > 0;
  const bool um = d.out_unit_major != 0;  // output projections stored [in, out]: the three GEMM forms rotate
  // Masked variant (Section 4.1, "Masked TwIST"): `sub` is a full-width subnet and the blocks that row `mask_row` of
  // `mask_plan` does not name are masked; the module scales are those of the masked widths.  Two ways, same results:
  //  - compact (struct Compact above): nothing is computed for masked blocks;
  //  - in place: they are computed at full width and zeroed where they enter the output projections (attention output
  //    columns, FFN activations) and where the gradient comes back through the same places, inside the kernels that produce
  //    those tensors.  The ordinary pass, with the same number of launches.
  // (twist_train_masked_compact chooses.)
  if (mask_plan) {
    for (int l = 0; l < d.n_layers; ++l)
      if (L.heads_sub[l] != d.n_heads || L.ffn_sub[l] != ctx->n_ffn_units())
        TW_FAIL(ctx, TWIST_ESHAPE, "masked pass: the subnet must hold every block of layer %d", l);
  }
  std::vector<int32_t> heads = L.heads_sub, ffn = L.ffn_sub;  // width of every layer as it is run
  std::vector<Compact> compact(d.n_layers);
  if (mask_plan && !forward_only && twist_train_masked_compact(ctx, mask_plan, B, N)) {
    for (int l = 0; l < d.n_layers; ++l) {
      heads[l] = mask_plan->at(l, TWIST_KIND_HEAD).n_sub;
      ffn[l] = mask_plan->at(l, TWIST_KIND_FFN).n_sub;
      compact_layout(d, mask_plan, l, compact[l]);
      compact[l].on = true;
    }
    carve(ctx, heads, ffn, mask_plan, B, N, ws, w);
  }
  const bool in_place = mask_plan && !compact[0].on;
  // per-block mask of layer l (device table: entry < 0 = block not kept), handed to the kernels that produce the attention
  // output, the FFN activation and their gradients; null in the ordinary pass
  auto keep_of = [&](int l, int kind) -> const int32_t * {
    if (!in_place) return nullptr;
    const PlanEntry &pe = mask_plan->at(l, kind);
    return pe.d_inv + (size_t)mask_row * pe.n_full;
  };
  auto kept = [&](int l, int kind, int full) { return mask_plan ? mask_plan->at(l, kind).n_sub : full; };
  const int scale_mode = mask_plan ? mask_plan->scale_mode : sub->plan->scale_mode;
  auto P = [&](const Slot &s) -> void * { return s.off < 0 ? nullptr : sub->params + s.off * es; };
  auto G = [&](const Slot &s) -> float * { return s.off < 0 ? nullptr : sub->grads + s.off; };
  // weight and gradient of layer l's tensor t as the pass uses them: in the subnet, or in the compact scratch
  auto PW = [&](int l, int t) -> void * {
    const Compact &c = compact[l];
    return c.on && c.off[t] >= 0 ? w.cw + c.off[t] * es : P(L.at(l, t));
  };
  auto GW = [&](int l, int t) -> float * {
    const Compact &c = compact[l];
    if (!c.on || c.off[t] < 0) return G(L.at(l, t));
    return c.off[t] >= c.bias_off ? w.cb + l * w.cb_stride + (c.off[t] - c.bias_off) : w.cg + c.off[t];
  };
  int gathered = -1;  // layer whose kept blocks the scratch holds
  auto gather_layer = [&](int l) -> twist_status {
    if (!compact[l].on || compact[l].elems == 0 || gathered == l) return TWIST_OK;
    const void *full[TWIST_N_LAYER_TENSORS];
    for (int t = 0; t < TWIST_N_LAYER_TENSORS; ++t) full[t] = P(L.at(l, t));
    gathered = l;
    return twist_gather_layer(ctx, mask_plan, l, mask_row, full, compact[l].off, w.cw);
  };
  // gradients of the tensors in `only` from the scratch to their full-width places
  auto expand = [&](hipStream_t st, int l, uint32_t only, const float *src, int64_t shift) -> twist_status {
    const Compact &c = compact[l];
    if (!c.on) return TWIST_OK;
    float *full[TWIST_N_LAYER_TENSORS];
    int64_t off[TWIST_N_LAYER_TENSORS];
    for (int t = 0; t < TWIST_N_LAYER_TENSORS; ++t) { full[t] = G(L.at(l, t)); off[t] = c.off[t] < 0 ? -1 : c.off[t] - shift; }
    return twist_expand_layer(ctx, st, mask_plan, l, mask_row, full, off, src, only);
  };
  auto gemm = [&](GemmLayout lay, int M, int Nn, int K, const void *A, int64_t lda, const void *Bm, int64_t ldb, void *out, int64_t ldc, int out_f32,
                  float alpha = 1.f, const void *bias = nullptr, const float *residual = nullptr) {
    GemmEpilogue e;
    e.alpha = alpha; e.bias = bias; e.residual = residual; e.out = out; e.out_f32 = out_f32;
    return twist_gemm(ctx, bf, lay, M, Nn, K, A, lda, Bm, ldb, ldc, e);
  };
  // Norm backward of norm layer `idx` (2l, 2l+1: the two norms of layer l; 2 n_layers: the final norm).  Its parameter
  // gradients are left as per-chunk partial sums in the layer's own block and summed for all layers by one launch at
  // the end of the pass, which takes 2 n_layers small kernels off the chain of dependent kernels.
  std::vector<ColReduce> reduce_items;
  // Per-chunk column sums behind the bias gradients, reduced with everything else at the end; layer l's block: FFN down and attention
  // output (the residual gradient's sums, formed by the norm backward that produces it), then FFN up, then q/k/v.
  const size_t sum_d = twist_colsum_partial_floats(T, D);
  auto down_sums = [&](int l) { return l >= 0 && L.at(l, TWIST_B_DOWN).off >= 0 ? w.bias_partial + (size_t)l * w.bias_partial_stride : nullptr; };
  auto out_sums = [&](int l) { return L.at(l, TWIST_BO).off >= 0 ? w.bias_partial + (size_t)l * w.bias_partial_stride + sum_d : nullptr; };
  // csum: where the column sums of the activation-type copy go (the next projection's bias gradient), or null.
  auto norm_bwd = [&](int idx, const void *dy, const float *x, const void *nw, int accumulate, void *dxb, float *dw, float *db, float *csum) {
    float *part = w.norm_partial + (size_t)idx * w.norm_partial_stride;
    reduce_items.push_back({part, dw, 2 * (int64_t)D, D, 1.f});
    if (db) reduce_items.push_back({part + D, db, 2 * (int64_t)D, D, 1.f});
    return twist_norm_bwd(ctx, bf, rms, dy, x, nw, w.stats[idx], w.dx, accumulate, dxb, dw, db, part, T, D, true, csum);
  };

  // ------------------------------------------------------------------------------------ forward
  if (lm) {
    TW_TRY(twist_embed_fwd(ctx, bf, static_cast<const int32_t *>(inputs), P(L.global[TWIST_TOK_EMBED]), P(L.global[TWIST_POS_EMBED]), w.xs[0], B, N, D,
                           d.vocab));
  } else {
    TW_TRY(twist_cast_in(ctx, bf, inputs, w.xs[0], (int64_t)T * D));
  }
  if (d.use_rope) TW_TRY(twist_rope_table(ctx, w.rope_tab, N, dh, d.rope_theta));

  for (int l = 0; l < d.n_layers; ++l) {
    const int Hs = heads[l], HD = Hs * dh, F = ffn[l] * d.ffn_granule;
    const float c_a = scale_mode ? sqrtf((float)d.n_heads / (float)kept(l, TWIST_KIND_HEAD, Hs)) : 1.f;
    const float c_f = scale_mode ? sqrtf((float)ctx->n_ffn_units() / (float)kept(l, TWIST_KIND_FFN, ffn[l])) : 1.f;
    const LayerBufs &b = w.layer[l];
    TW_TRY(gather_layer(l));
    TW_TRY(twist_norm_fwd(ctx, bf, rms, w.xs[2 * l], P(L.at(l, TWIST_NORM1_W)), P(L.at(l, TWIST_NORM1_B)), b.h1, w.stats[2 * l], T, D, d.norm_eps));
    TW_TRY(gemm(GEMM_NT, T, 3 * HD, D, b.h1, D, PW(l, TWIST_WQ), D, b.qkv, 3 * HD, 0, 1.f, PW(l, TWIST_BQ)));
    if (d.use_rope) TW_TRY(twist_rope_apply(ctx, bf, b.qkv, w.rope_tab, B, N, Hs, dh, 1.f));
    TW_TRY(twist_attention_fwd(ctx, bf, b.qkv, b.o, forward_only ? nullptr : b.o32, b.lse, B, N, Hs, dh, keep_of(l, TWIST_KIND_HEAD)));
    if (um) TW_TRY(gemm(GEMM_NN, T, D, HD, b.o, HD, PW(l, TWIST_WO), D, w.xs[2 * l + 1], D, 1, c_a, P(L.at(l, TWIST_BO)), w.xs[2 * l]));
    else TW_TRY(gemm(GEMM_NT, T, D, HD, b.o, HD, PW(l, TWIST_WO), HD, w.xs[2 * l + 1], D, 1, c_a, P(L.at(l, TWIST_BO)), w.xs[2 * l]));
    TW_TRY(twist_norm_fwd(ctx, bf, rms, w.xs[2 * l + 1], P(L.at(l, TWIST_NORM2_W)), P(L.at(l, TWIST_NORM2_B)), b.h2, w.stats[2 * l + 1], T, D, d.norm_eps));
    const int w1 = nf == 2 ? TWIST_W_GATE : TWIST_W_UP;
    if (nf == 1 && !in_place) {  // ungated: the projection applies it
      GemmEpilogue e;
      e.bias = PW(l, TWIST_B_UP); e.out = b.gu; e.act_out = b.a; e.act = d.act; e.act_only = forward_only;
      TW_TRY(twist_gemm(ctx, bf, GEMM_NT, T, F, D, b.h2, D, PW(l, w1), D, F, e));
    } else {
      TW_TRY(gemm(GEMM_NT, T, nf * F, D, b.h2, D, PW(l, w1), D, b.gu, nf * F, 0, 1.f, PW(l, TWIST_B_UP)));
      TW_TRY(twist_act_fwd(ctx, bf, d.act, b.gu, b.a, T, F, keep_of(l, TWIST_KIND_FFN), d.ffn_granule));
    }
    if (um) TW_TRY(gemm(GEMM_NN, T, D, F, b.a, F, PW(l, TWIST_W_DOWN), D, w.xs[2 * l + 2], D, 1, c_f, P(L.at(l, TWIST_B_DOWN)), w.xs[2 * l + 1]));
    else TW_TRY(gemm(GEMM_NT, T, D, F, b.a, F, PW(l, TWIST_W_DOWN), F, w.xs[2 * l + 2], D, 1, c_f, P(L.at(l, TWIST_B_DOWN)), w.xs[2 * l + 1]));
  }

  // ------------------------------------------------------------------------------------ loss and its gradient
  float *x_last = w.xs[2 * d.n_layers];
  if (lm) {
    const int V = d.vocab;
    const Slot &wout = d.tied_head ? L.global[TWIST_TOK_EMBED] : L.global[TWIST_LM_HEAD];
    TW_TRY(twist_norm_fwd(ctx, bf, rms, x_last, P(L.global[TWIST_FINAL_NORM_W]), P(L.global[TWIST_FINAL_NORM_B]), w.hf, w.stats[2 * d.n_layers], T, D,
                          d.norm_eps));
    int blocks = 0;  // of the loss parts that the projection leaves instead of the logits
    {
      GemmEpilogue e;
      e.out = w.logits;
      if (forward_only) {
        e.targets = static_cast<const int32_t *>(targets);
        e.loss_parts = static_cast<float *>(w.logits);  // (8 bytes for 64 columns or more: they fit the logits' place)
        e.target_logit = w.rowloss;
        e.loss_blocks = &blocks;
      }
      TW_TRY(twist_gemm(ctx, bf, GEMM_NT, T, V, D, w.hf, D, P(wout), D, w.ld_logits, e));
    }
    if (blocks) return twist_ce_parts(ctx, static_cast<const float *>(w.logits), blocks, w.rowloss, loss_dev, T);
    TW_TRY(twist_ce_fwd_bwd(ctx, bf, w.logits, w.ld_logits, static_cast<const int32_t *>(targets), w.rowloss, loss_dev, T, V, !forward_only));
    if (forward_only) return TWIST_OK;
    // projection weight gradient, then the gradient flowing back into the final norm
    TW_TRY(gemm(GEMM_TN, V, D, T, w.logits, w.ld_logits, w.hf, D, G(wout), D, 1));
    {
      // gradient of the final normed input: few output tiles ([T, d_model]) and a contraction as long as the vocabulary, so
      // it may be cut along the vocabulary like the weight gradients (the scratch is free here: the second stream's
      // projections of this pass have not started, those of the previous pass were joined before it returned)
      GemmEpilogue e;
      e.out = w.dh; e.out_f32 = 0;
      e.splitk_ws = w.splitk; e.splitk_floats = kSplitkFloats;
      TW_TRY(twist_gemm(ctx, bf, GEMM_NN, T, D, V, w.logits, w.ld_logits, P(wout), D, D, e));
    }
    TW_TRY(norm_bwd(2 * d.n_layers, w.dh, x_last, P(L.global[TWIST_FINAL_NORM_W]), 0, w.dxb, G(L.global[TWIST_FINAL_NORM_W]),
                    G(L.global[TWIST_FINAL_NORM_B]), down_sums(d.n_layers - 1)));
  } else {
    TW_TRY(twist_mse_fwd_bwd(ctx, bf, x_last, targets, w.dx, w.dxb, w.rowloss, loss_dev, (int64_t)T * D));
    if (forward_only) return TWIST_OK;
    if (float *sums = down_sums(d.n_layers - 1)) TW_TRY(twist_colsum(ctx, bf, w.dxb, D, 1.f, nullptr, sums, T, D, true));
  }

  // ------------------------------------------------------------------------------------ backward through the layers
  SideStream side(ctx);
  int64_t sum_heads = 0, sum_ffn = 0;
  for (int l = 0; l < d.n_layers; ++l) { sum_heads += heads[l]; sum_ffn += ffn[l]; }
  TW_TRY(side.init(T, D, (int)(sum_heads * dh / d.n_layers), (int)(sum_ffn * d.ffn_granule / d.n_layers), nf));
  // Weight gradients wait in `grads` and run together
  std::vector<WeightGrad> grads;
  uint32_t grads_of = 0;
  auto wgrad = [&](int M, int Nn, const void *A, int64_t lda, const void *Bm, int64_t ldb, float *out, float alpha, uint32_t tensors) {
    grads.push_back({M, Nn, A, lda, Bm, ldb, out, alpha});
    grads_of |= tensors;
  };
  auto run_wgrads = [&](int l, int slot) -> twist_status {
    TW_TRY(side.fork(slot));
    TW_TRY(twist_weight_grads(ctx, bf, (int)grads.size(), grads.data(), T, w.splitk, kSplitkFloats, side.stream()));  // (one scratch: one stream)
    TW_TRY(expand(side.stream(), l, grads_of, w.cg, 0));
    TW_TRY(side.done(slot));
    grads.clear();
    grads_of = 0;
    return TWIST_OK;
  };
  void *gx = w.dxb, *gx_other = w.dxb2;  // gradient of the residual stream in activation type: current, spare
  for (int l = d.n_layers - 1; l >= 0; --l) {
    const int Hs = heads[l], HD = Hs * dh, F = ffn[l] * d.ffn_granule;
    const float c_a = scale_mode ? sqrtf((float)d.n_heads / (float)kept(l, TWIST_KIND_HEAD, Hs)) : 1.f;
    const float c_f = scale_mode ? sqrtf((float)ctx->n_ffn_units() / (float)kept(l, TWIST_KIND_FFN, ffn[l])) : 1.f;
    const LayerBufs &b = w.layer[l];
    TW_TRY(gather_layer(l));
    const int w1 = nf == 2 ? TWIST_W_GATE : TWIST_W_UP;
    // FFN branch: y = c_f (a W_down^T + b_down)
    // bias gradients of the partitioned biases: per-chunk column sums now, reduced with everything else at the end
    float *bias_part = w.bias_partial + (size_t)l * w.bias_partial_stride + 2 * sum_d;
    auto bias_sums = [&](float *out, int n) {
      float *part = bias_part;
      bias_part += twist_colsum_partial_floats(T, n);
      reduce_items.push_back({part, out, (int64_t)n, n, 1.f});
      return part;
    };
    if (float *sums = down_sums(l)) reduce_items.push_back({sums, G(L.at(l, TWIST_B_DOWN)), (int64_t)D, D, c_f});
    if (um) wgrad(F, D, b.a, F, gx, D, GW(l, TWIST_W_DOWN), c_f, 1u << TWIST_W_DOWN);
    else wgrad(D, F, gx, D, b.a, F, GW(l, TWIST_W_DOWN), c_f, 1u << TWIST_W_DOWN);
    if (!side.whole && !side.ffn_pair) TW_TRY(run_wgrads(l, 0));
    if (um) TW_TRY(gemm(GEMM_NT, T, F, D, gx, D, PW(l, TWIST_W_DOWN), D, w.da, F, 0, c_f));
    else TW_TRY(gemm(GEMM_NN, T, F, D, gx, D, PW(l, TWIST_W_DOWN), F, w.da, F, 0, c_f));
    TW_TRY(side.wait_done(1));
    TW_TRY(twist_act_bwd(ctx, bf, d.act, b.gu, w.da, w.dgu, T, F, keep_of(l, TWIST_KIND_FFN), d.ffn_granule,
                         L.at(l, TWIST_B_UP).off >= 0 ? bias_sums(GW(l, TWIST_B_UP), nf * F) : nullptr));
    wgrad(nf * F, D, w.dgu, nf * F, b.h2, D, GW(l, w1), 1.f, 1u << TWIST_W_GATE | 1u << TWIST_W_UP);
    if (!side.whole) TW_TRY(run_wgrads(l, 1));
    TW_TRY(gemm(GEMM_NN, T, D, nf * F, w.dgu, nf * F, PW(l, w1), D, w.dh, D, 0));
    TW_TRY(side.wait_done(side.attn_pair ? 3 : 2));
    TW_TRY(norm_bwd(2 * l + 1, w.dh, w.xs[2 * l + 1], P(L.at(l, TWIST_NORM2_W)), 1, gx_other, G(L.at(l, TWIST_NORM2_W)), G(L.at(l, TWIST_NORM2_B)), out_sums(l)));
    // attention branch: y = c_a (o C_attn^T + b_o)
    if (float *sums = out_sums(l)) reduce_items.push_back({sums, G(L.at(l, TWIST_BO)), (int64_t)D, D, c_a});
    if (um) wgrad(HD, D, b.o, HD, gx_other, D, GW(l, TWIST_WO), c_a, 1u << TWIST_WO);
    else wgrad(D, HD, gx_other, D, b.o, HD, GW(l, TWIST_WO), c_a, 1u << TWIST_WO);
    if (!side.whole && !side.attn_pair) TW_TRY(run_wgrads(l, 2));
    if (um) TW_TRY(gemm(GEMM_NT, T, HD, D, gx_other, D, PW(l, TWIST_WO), D, w.dout, HD, 0, c_a));
    else TW_TRY(gemm(GEMM_NN, T, HD, D, gx_other, D, PW(l, TWIST_WO), HD, w.dout, HD, 0, c_a));
    TW_TRY(side.wait_done(3));
    TW_TRY(twist_attention_bwd(ctx, bf, b.qkv, bf ? b.o32 : static_cast<const float *>(b.o), w.dout, b.lse, w.delta, w.dqkv, B, N, Hs, dh, d.use_rope ? w.rope_tab : nullptr,
                               keep_of(l, TWIST_KIND_HEAD)));
    if (L.at(l, TWIST_BQ).off >= 0) TW_TRY(twist_colsum(ctx, bf, w.dqkv, 3 * HD, 1.f, nullptr, bias_sums(GW(l, TWIST_BQ), 3 * HD), T, 3 * HD, true));
    wgrad(3 * HD, D, w.dqkv, 3 * HD, b.h1, D, GW(l, TWIST_WQ), 1.f, 1u << TWIST_WQ | 1u << TWIST_WK | 1u << TWIST_WV);
    TW_TRY(run_wgrads(l, 3));
    TW_TRY(gemm(GEMM_NN, T, D, 3 * HD, w.dqkv, 3 * HD, PW(l, TWIST_WQ), D, w.dh, D, 0));
    TW_TRY(side.wait_done(side.ffn_pair ? 1 : 0));
    TW_TRY(norm_bwd(2 * l, w.dh, w.xs[2 * l], P(L.at(l, TWIST_NORM1_W)), 1, gx, G(L.at(l, TWIST_NORM1_W)), G(L.at(l, TWIST_NORM1_B)), down_sums(l - 1)));
  }
  TW_TRY(twist_col_reduce_batch(ctx, reduce_items.data(), (int)reduce_items.size(), T));
  if (d.has_bias)
    for (int l = 0; l < d.n_layers; ++l)
      TW_TRY(expand(nullptr, l, 1u << TWIST_BQ | 1u << TWIST_BK | 1u << TWIST_BV | 1u << TWIST_B_UP, w.cb + l * w.cb_stride, compact[l].bias_off));
  for (int i = 0; i < 4; ++i) TW_TRY(side.wait_done(i));  // join: the caller's stream sees the whole pass
  (void)gx_other;

  if (lm) {
    // token embedding: rows used by this batch receive dx (on top of the projection gradient when tied)
    const Slot &te = L.global[TWIST_TOK_EMBED];
    if (!d.tied_head) TW_TRY(twist_zero_f32(ctx, G(te), (int64_t)te.rows * te.cols));
    TW_TRY(twist_embed_bwd(ctx, static_cast<const int32_t *>(inputs), w.dx, G(te), G(L.global[TWIST_POS_EMBED]), B, N, D));
    const Slot &pe = L.global[TWIST_POS_EMBED];
    if (pe.off >= 0 && N < pe.rows) TW_TRY(twist_zero_f32(ctx, G(pe) + (size_t)N * D, (int64_t)(pe.rows - N) * D));
  }
  return TWIST_OK;
}

extern "C" twist_status twist_backward_schedule(twist_ctx *ctx, int32_t tokens, int32_t head_columns, int32_t ffn_columns, int32_t chosen[4]) {
  if (!ctx || !chosen) TW_FAIL(ctx, TWIST_EINVAL, "twist_backward_schedule: null argument");
  if (tokens < 1 || head_columns < 1 || ffn_columns < 1) TW_FAIL(ctx, TWIST_EINVAL, "twist_backward_schedule: bad size");
  Schedule s;
  s.choose(ctx->d.dtype == TWIST_BF16, tokens, ctx->d.d_model, head_columns, ffn_columns, ctx->d.act == TWIST_ACT_SWIGLU ? 2 : 1);
  chosen[0] = s.whole; chosen[1] = s.ffn_pair; chosen[2] = s.attn_pair; chosen[3] = !s.whole && ctx->overlap;
  return TWIST_OK;
}

twist_status twist_train_step(twist_ctx *ctx, twist_subnet *sub, const twist_opt_desc *opt) {
  if (!sub->grads) TW_FAIL(ctx, TWIST_ESHAPE, "step: subnet was extracted without gradient storage");
  const SubLayout &L = sub->plan->layout;
  const int bf = ctx->d.dtype == TWIST_BF16;
  if (opt->kind == TWIST_OPT_SGD) return twist_sgd(ctx, bf, sub->params, sub->master, sub->grads, L.n_total, opt->lr);
  if (opt->kind == TWIST_OPT_ADAMW) {
    if (!sub->adam_m) TW_FAIL(ctx, TWIST_ESHAPE, "step: AdamW needs a subnet extracted with TWIST_STORE_ADAMW");
    sub->step_count += 1;
    return twist_adamw(ctx, bf, sub->params, sub->master, sub->grads, sub->adam_m, sub->adam_v, L.n_total, L.n_matrix, opt->lr, opt->beta1, opt->beta2,
                       opt->eps, opt->weight_decay, sub->step_count);
  }
  TW_FAIL(ctx, TWIST_EINVAL, "step: unknown optimizer %d", opt->kind);
}
