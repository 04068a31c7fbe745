"""Kernel-level parity of the memory-bound steps of the subnet pass (norms, rotary positions, activations, loss,
embedding, the Masked-TwIST masks), each against the checker's unrounded fp64 function on identical inputs:
<= 5e-3 where a bf16 result is stored (one rounding: about 1.1e-3), <= 1e-4 for fp32 results of either model type."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import synth_inputs as si
from helpers import rel_fro, to_numpy
from oracle import model as omodel

pytestmark = pytest.mark.gpu

BF, F32 = "bf16", "f32"


def _snap(a, dtype):
    return si.to_bf16_grid(a) if dtype == BF else np.asarray(a, np.float32).astype(np.float64)


def _dev(a, dtype=None):
    t = torch.tensor(np.ascontiguousarray(a), dtype=torch.float64)
    return t.to({BF: torch.bfloat16, F32: torch.float32, None: torch.float32}[dtype]).cuda().contiguous()


def _tol(dtype):
    return 5e-3 if dtype == BF else 1e-4


# d_model: 256, 768, 2048, 4096 take the kernels that hold a row in registers (1, 3, 8, 16 vectors per lane), 200 the
# general kernels; T = 37 leaves a ragged last chunk of 16 rows
@pytest.mark.parametrize("dtype", [BF, F32])
@pytest.mark.parametrize("kind,D,T", [("rms", 256, 37), ("ln", 256, 64), ("ln", 768, 37), ("rms", 2048, 50), ("rms", 4096, 33), ("ln", 200, 37),
                                       ("rms", 200, 16), ("ln", 1024, 19)])
def test_norm_forward_and_backward(lib, dtype, kind, D, T):
    cfg = si.ModelCfg(d_model=D, n_heads=1, d_head=8, d_ff=8, norm=kind, dtype=dtype)
    ctx = lib.Context(lib.desc_from_cfg(cfg))
    x = np.asarray(si.normal(D + T, "x", (T, D), 1.5) + 0.3, np.float32).astype(np.float64)      # the residual stream is fp32
    w, b = _snap(1.0 + si.normal(D, "w", (D,), 0.2), dtype), _snap(si.normal(D, "b", (D,), 0.2), dtype)
    dy = _snap(si.normal(T, "dy", (T, D)), dtype)
    bb = b if kind == "ln" else None
    y, stats, (dx, dxb, dw, db) = ctx.twist_norm_raw(_dev(x), _dev(w, dtype), _dev(bb, dtype) if bb is not None else None, _dev(dy, dtype))
    torch.cuda.synchronize()
    want_y, cache = omodel.norm_fwd(x, w, bb, kind, cfg.norm_eps)
    want_dx, want_dw, want_db = omodel.norm_bwd(dy, w, cache, kind)
    assert rel_fro(to_numpy(y), want_y) <= _tol(dtype)
    np.testing.assert_allclose(to_numpy(stats[:, 1]), cache[1][:, 0], rtol=1e-5)
    assert rel_fro(to_numpy(dx), want_dx) <= 1e-4                      # fp32 result in both model types
    assert rel_fro(to_numpy(dxb), want_dx) <= _tol(dtype)
    assert rel_fro(to_numpy(dw), want_dw) <= 1e-4
    if kind == "ln":
        assert rel_fro(to_numpy(db), want_db) <= 1e-4


# widths that fill the last vector of 256 columns, have one lane in it or leave most of it empty, in every kernel: a wave per row (1 to 4 vectors, with
# four and with eight waves to a chunk of 16 rows; 6 and 8 vectors) and four waves per row (beyond 2048); ragged last chunks
@pytest.mark.parametrize("dtype", [BF, F32])
@pytest.mark.parametrize("kind,D,T", [("ln", 4, 5), ("rms", 12, 4097), ("ln", 252, 4100), ("ln", 260, 40), ("rms", 516, 33), ("ln", 1020, 4099), ("ln", 1284, 50), ("rms", 1536, 20),
                                       ("ln", 1928, 35), ("ln", 2052, 18), ("rms", 3072, 33), ("ln", 3076, 19), ("ln", 4096, 33), ("rms", 4100, 17), ("ln", 70, 20)])
def test_norm_of_any_width(lib, dtype, kind, D, T):
    test_norm_forward_and_backward(lib, dtype, kind, D, T)


@pytest.mark.parametrize("dtype", [BF, F32])
@pytest.mark.parametrize("dh,Hs,B,N", [(128, 2, 2, 48), (64, 3, 1, 40), (6, 5, 2, 9)])
def test_rotary_positions(lib, dtype, dh, Hs, B, N):
    cfg = si.ModelCfg(arch="llama", d_model=64, n_heads=Hs, d_head=dh, d_ff=8, rope=True, dtype=dtype)
    ctx = lib.Context(lib.desc_from_cfg(cfg))
    qkv = _snap(si.normal(dh, "qkv", (B * N, 3 * Hs * dh)), dtype)
    cos, sin = omodel.rope_tables(N, dh, cfg.rope_theta)
    for sign in (1.0, -1.0):
        t = _dev(qkv, dtype)
        ctx.twist_rope_raw(t, B, N, Hs, sign)
        torch.cuda.synchronize()
        got = to_numpy(t)
        heads = qkv.reshape(B, N, 3 * Hs, dh)
        want = heads.copy()
        want[:, :, :2 * Hs] = omodel.rope_apply(heads[:, :, :2 * Hs], cos, sin, sign)       # q and k heads turn, v stays
        assert rel_fro(got, want.reshape(B * N, -1)) <= _tol(dtype)
        assert np.array_equal(got.reshape(B, N, 3 * Hs, dh)[:, :, 2 * Hs:], heads[:, :, 2 * Hs:])


@pytest.mark.parametrize("dtype", [BF, F32])
@pytest.mark.parametrize("act,T,F,unit", [("swiglu", 37, 352, 1), ("swiglu", 5, 44, 4), ("gelu_tanh", 37, 512, 1), ("gelu_tanh", 9, 35, 5),
                                           ("relu", 37, 512, 64), ("relu", 9, 35, 7), ("relu", 3, 12, 1)])
def test_activation_forward_backward_and_neuron_mask(lib, dtype, act, T, F, unit):
    """Without a mask: a = f(u), dgu = da f'(u).  With the Masked-TwIST mask (Section 4.1, y = M * f(x)): masked blocks give
    exact zeros in a and dgu, kept blocks the unmasked values bit for bit."""
    cfg = si.ModelCfg(d_model=64, n_heads=1, d_head=8, d_ff=F, ffn_granule=unit, act=act, has_bias=act != "swiglu", dtype=dtype)
    ctx = lib.Context(lib.desc_from_cfg(cfg))
    nf = 2 if act == "swiglu" else 1
    gu = _snap(si.normal(F, "gu", (T, nf * F), 1.5), dtype)
    da = _snap(si.normal(T, "da", (T, F)), dtype)
    a, dgu = ctx.twist_act_raw(_dev(gu, dtype), F, _dev(da, dtype))
    torch.cuda.synchronize()
    if act == "swiglu":
        g, u = gu[:, :F], gu[:, F:]
        want_a = omodel.swiglu_fwd(g, u)
        dg, du = omodel.swiglu_bwd(g, u, da)
        want_d = np.concatenate([dg, du], axis=1)
    else:
        want_a, want_d = omodel.act_fwd(gu, act), da * omodel.act_bwd(gu, act)
    assert rel_fro(to_numpy(a), want_a) <= _tol(dtype), rel_fro(to_numpy(a), want_a)
    assert rel_fro(to_numpy(dgu), want_d) <= _tol(dtype), rel_fro(to_numpy(dgu), want_d)
    rng = np.random.default_rng(F + unit)
    keep_np = np.where(rng.random(F // unit) < 0.5, -1, rng.integers(0, 100, F // unit)).astype(np.int32)
    keep_np[0], keep_np[-1] = -1, 3
    keep = torch.tensor(keep_np).cuda()
    am, dm = ctx.twist_act_raw(_dev(gu, dtype), F, _dev(da, dtype), keep=keep, unit=unit)
    torch.cuda.synchronize()
    on = np.repeat(keep_np >= 0, unit)
    am, dm, a, dgu = (to_numpy(t) for t in (am, dm, a, dgu))
    assert not am[:, ~on].any() and np.array_equal(am[:, on], a[:, on])
    on2 = np.tile(on, nf)
    assert not dm[:, ~on2].any() and np.array_equal(dm[:, on2], dgu[:, on2])


# vocabulary: 515 and 1003 (rows held in registers, 4 vectors per lane), 32000 (16 vectors), 33001 to 65536 (16 vectors, 512 threads), 70001 (re-read kernel); the
# row stride is the vocabulary rounded up to 8, as in the training pass; 301 with fp32 takes the general kernel
@pytest.mark.parametrize("dtype,V,T", [(BF, 515, 37), (BF, 1003, 8), (BF, 32000, 6), (BF, 33001, 5), (BF, 50257, 3), (BF, 65536, 2), (BF, 70001, 2), (F32, 301, 37), (F32, 1003, 5)])
def test_cross_entropy_loss_and_gradient(lib, dtype, V, T):
    cfg = si.ModelCfg(d_model=64, n_heads=1, d_head=8, d_ff=8, vocab=V, dtype=dtype)
    ctx = lib.Context(lib.desc_from_cfg(cfg))
    ld = (V + 7) // 8 * 8
    logits = _snap(si.normal(V, "logits", (T, V), 2.0), dtype)
    tgt = si.tokens_uniform(V, 1, T - 1, V)[0].astype(np.int32)
    tgt[0], tgt[-1] = V - 1, 0
    padded = np.full((T, ld), 7.0)                                        # the padding must not enter the sums
    padded[:, :V] = logits
    t = _dev(padded, dtype)
    loss, rowloss = ctx.twist_ce_raw(t, torch.tensor(tgt).cuda())
    torch.cuda.synchronize()
    want_loss, want_d = omodel.cross_entropy(logits[None], tgt[None].astype(np.int64))
    assert abs(loss.item() - want_loss) <= 1e-5 * abs(want_loss), (loss.item(), want_loss)
    got = to_numpy(t)
    assert rel_fro(got[:, :V], want_d[0]) <= _tol(dtype), rel_fro(got[:, :V], want_d[0])
    if dtype == BF:
        assert not got[:, V:].any()                                       # padding columns feed the next projection as zeros
    np.testing.assert_allclose(to_numpy(rowloss).mean(), want_loss, rtol=1e-5)


# fp32 rows held in registers: 4 vectors per lane of 256 threads, 16 of 256, of 512 and of 1024, and the re-read kernel beyond 65536; strides of the
# vocabulary rounded up to 8, vocabularies that end in a vector, at it and before it
@pytest.mark.parametrize("V,T", [(1, 2), (4, 3), (4093, 5), (4097, 4), (16383, 3), (16385, 3), (32768, 2), (32775, 2), (50257, 3), (65534, 2), (65537, 2)])
@pytest.mark.parametrize("odd", [None, float("inf"), float("nan"), torch.finfo(torch.float32).min])
def test_fp32_cross_entropy_at_the_edges_of_its_kernels(lib, V, T, odd):
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=1, d_head=8, d_ff=8, vocab=V, dtype=F32)))
    x = torch.randn(T, (V + 7) // 8 * 8, generator=torch.Generator().manual_seed(V)) * 3
    x[:, V:] = float("nan")                                               # the padding must not enter the sums
    if odd is not None:
        x[0, V // 2] = odd
    tgt = torch.tensor([V - 1] + [(7919 * i) % V for i in range(1, T)], dtype=torch.int32)
    t = x.cuda()
    loss, rowloss = ctx.twist_ce_raw(t, tgt.cuda())
    torch.cuda.synchronize()
    z = x[:, :V].double()
    rows = torch.arange(T)
    want_loss, want = torch.logsumexp(z, 1) - z[rows, tgt.long()], torch.softmax(z, 1)
    want[rows, tgt.long()] -= 1
    sound = torch.isfinite(want).all(1)
    rowloss, got = rowloss.cpu().double(), t.cpu().double() * T
    assert not torch.isfinite(rowloss[~sound]).any()
    # exponentials of relative error 2^-22 and 2^-24 |x - lse| (at most 30) of their argument; loss: an fp32 sum and difference of values below 32
    torch.testing.assert_close(rowloss[sound], want_loss[sound], rtol=2e-6, atol=4e-6)
    torch.testing.assert_close(got[sound][:, :V], want[sound], rtol=1e-5, atol=1e-6)
    assert not got[sound][:, V:].any()


@pytest.mark.parametrize("dtype", [BF, F32])
@pytest.mark.parametrize("positions", [True, False])
def test_embedding_forward_and_backward(lib, dtype, positions):
    V, D, B, N, P = 53, 72, 3, 10, 12
    cfg = si.ModelCfg(d_model=D, n_heads=1, d_head=8, d_ff=8, vocab=V, max_seq=P, dtype=dtype)
    ctx = lib.Context(lib.desc_from_cfg(cfg))
    E, Pz = _snap(si.normal(1, "E", (V, D)), dtype), _snap(si.normal(2, "P", (P, D)), dtype)
    tok = si.tokens_uniform(V, B, N - 1, 5).astype(np.int32)
    tok[0, :3] = 7                                                          # a repeated token: its gradient rows add up
    dx = np.asarray(si.normal(3, "dx", (B, N, D)), np.float32).astype(np.float64)
    x, d_tok, d_pos = ctx.twist_embed_raw(torch.tensor(tok).cuda(), _dev(E, dtype), _dev(Pz, dtype) if positions else None, _dev(dx.reshape(B * N, D)))
    torch.cuda.synchronize()
    want_x = omodel.embed_fwd(tok.astype(np.int64), E, Pz if positions else None)
    assert rel_fro(to_numpy(x), want_x.reshape(B * N, D)) <= 1e-6          # exact: a copy and at most one fp32 add
    dE = np.zeros((V, D))
    dP = omodel.embed_bwd(tok.astype(np.int64), dx, dE, P if positions else None)
    assert rel_fro(to_numpy(d_tok), dE) <= 1e-6
    if positions:
        assert rel_fro(to_numpy(d_pos), dP[:N]) <= 1e-6


@pytest.mark.parametrize("dtype,dh,N,choice", [(BF, 128, 256, {}), (BF, 128, 128, {"staged_attention": True}), (BF, 64, 128, {}),
                                               (BF, 32, 40, {}), (BF, 128, 128, {"plain_only": True}), (F32, 16, 37, {}),
                                               # one, three and five key blocks: the dK/dV kernel pairs key blocks, the middle one stays single
                                               (BF, 128, 128, {}), (BF, 128, 384, {}), (BF, 128, 640, {})])
def test_attention_head_mask(lib, dtype, dh, N, choice):
    """Masked TwIST's head mask inside the attention kernels (Section 4.1): a masked head's output and its q, k, v gradients
    are exact zeros, the kept heads' results are bit-identical to the unmasked call, in every kernel family (direct-to-LDS,
    register-staged, plain)."""
    Hs, B = 4, 2
    cfg = si.ModelCfg(d_model=64, n_heads=Hs, d_head=dh, d_ff=8, dtype=dtype, max_seq=N)
    ctx = lib.Context(lib.desc_from_cfg(cfg))
    ctx.twist_set_kernel_choice(**choice)
    qkv = _dev(_snap(si.normal(dh + N, "qkv", (B * N, 3 * Hs * dh)), dtype), dtype)
    dout = _dev(_snap(si.normal(N, "dout", (B * N, Hs * dh)), dtype), dtype)
    o, lse, dqkv = ctx.twist_attention_raw(qkv, dout, B, N, Hs)
    keep_np = np.array([5, -1, 0, -1], np.int32)
    om, lsem, dm = ctx.twist_attention_raw(qkv, dout, B, N, Hs, keep=torch.tensor(keep_np).cuda())
    torch.cuda.synchronize()
    o, om = to_numpy(o).reshape(B * N, Hs, dh), to_numpy(om).reshape(B * N, Hs, dh)
    d, dm = to_numpy(dqkv).reshape(B * N, 3, Hs, dh), to_numpy(dm).reshape(B * N, 3, Hs, dh)
    on = keep_np >= 0
    assert not om[:, ~on].any() and not dm[:, :, ~on].any()
    assert np.array_equal(om[:, on], o[:, on]) and np.array_equal(dm[:, :, on], d[:, :, on])
    assert o[:, ~on].any() and d[:, :, ~on].any()
    # and the unmasked results are the checker's attention (forward and backward) on the same inputs
    q, k, v = (to_numpy(qkv).reshape(B, N, 3, Hs, dh)[:, :, i] for i in range(3))
    want_o, p = omodel.attention_fwd(q, k, v)
    assert rel_fro(o.reshape(B, N, Hs, dh), want_o) <= _tol(dtype)
    wdq, wdk, wdv = omodel.attention_bwd(p, q, k, v, to_numpy(dout).reshape(B, N, Hs, dh))
    for i, want in enumerate((wdq, wdk, wdv)):
        assert rel_fro(d[:, i].reshape(B, N, Hs, dh), want) <= _tol(dtype), (i, rel_fro(d[:, i].reshape(B, N, Hs, dh), want))


@pytest.mark.parametrize("dh,N,choice", [(128, 256, {}), (128, 384, {}), (128, 128, {"staged_attention": True}), (64, 128, {}), (32, 40, {})])
def test_attention_backward_through_rotary_positions(lib, dh, N, choice):
    """The q and k gradients turned back through the rotary embedding (inside the direct-to-LDS kernels, by a separate
    rotation behind the others): the checker's attention backward followed by the inverse rotation."""
    Hs, B = 2, 2
    cfg = si.ModelCfg(arch="llama", d_model=64, n_heads=Hs, d_head=dh, d_ff=8, rope=True, dtype=BF, max_seq=N)
    ctx = lib.Context(lib.desc_from_cfg(cfg))
    ctx.twist_set_kernel_choice(**choice)
    qkv = _dev(_snap(si.normal(dh, "qkv", (B * N, 3 * Hs * dh)), BF), BF)
    dout = _dev(_snap(si.normal(N, "dout", (B * N, Hs * dh)), BF), BF)
    o, lse, dqkv = ctx.twist_attention_raw(qkv, dout, B, N, Hs, rope_backward=True)
    torch.cuda.synchronize()
    q, k, v = (to_numpy(qkv).reshape(B, N, 3, Hs, dh)[:, :, i] for i in range(3))
    _, p = omodel.attention_fwd(q, k, v)
    dq, dk, dv = omodel.attention_bwd(p, q, k, v, to_numpy(dout).reshape(B, N, Hs, dh))
    cos, sin = omodel.rope_tables(N, dh, cfg.rope_theta)
    want = (omodel.rope_apply(dq, cos, sin, -1.0), omodel.rope_apply(dk, cos, sin, -1.0), dv)
    got = to_numpy(dqkv).reshape(B, N, 3, Hs, dh)
    for i in range(3):
        assert rel_fro(got[:, :, i], want[i]) <= 5e-3, (i, rel_fro(got[:, :, i], want[i]))


# lengths that are no multiple of 128, and 32-wide heads, take the fp32-arithmetic tiles: one row, a partial and a full block of 32 rows,
# more tiles than waves, a ragged last one
@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("N", [1, 31, 33, 64, 65, 127, 129, 200, 321])
def test_attention_of_any_length(lib, dh, N):
    Hs, B = 3, 2
    cfg = si.ModelCfg(arch="llama", d_model=64, n_heads=Hs, d_head=dh, d_ff=8, rope=True, dtype=BF, max_seq=N)
    ctx = lib.Context(lib.desc_from_cfg(cfg))
    qkv = _dev(_snap(si.normal(dh + N, "qkv", (B * N, 3 * Hs * dh)), BF), BF)
    dout = _dev(_snap(si.normal(N, "dout", (B * N, Hs * dh)), BF), BF)
    o, lse, dqkv = ctx.twist_attention_raw(qkv, dout, B, N, Hs, rope_backward=True)
    torch.cuda.synchronize()
    q, k, v = (to_numpy(qkv).reshape(B, N, 3, Hs, dh)[:, :, i] for i in range(3))
    g = to_numpy(dout).reshape(B, N, Hs, dh)
    want_o, p = omodel.attention_fwd(q, k, v)
    assert rel_fro(to_numpy(o).reshape(B, N, Hs, dh), want_o) <= 5e-3
    dq, dk, dv = omodel.attention_bwd(p, q, k, v, g)
    cos, sin = omodel.rope_tables(N, dh, cfg.rope_theta)
    want = (omodel.rope_apply(dq, cos, sin, -1.0), omodel.rope_apply(dk, cos, sin, -1.0), dv)
    got = to_numpy(dqkv).reshape(B, N, 3, Hs, dh)
    for i in range(3):
        # dq and dk of a sequence of one are zero in exact arithmetic (one probability of 1): fp32 rounding of dp - delta is left,
        # 1e-7 of |dO| |v| |k|
        assert np.linalg.norm(got[:, :, i] - want[i]) <= 5e-3 * np.linalg.norm(want[i]) + 1e-5 * np.linalg.norm(g) * dh, i


# probabilities stay fp32 there: what is left is the results' own rounding to bf16, at most 2^-9 per value and, over the values, the
# root mean square of a uniform error in a binade, 1.66e-3 (with probabilities in bf16 it measures 2.0e-3, gradients 2.4e-3)
@pytest.mark.parametrize("dh,N", [(128, 200), (64, 333), (32, 256), (36, 100)])
def test_attention_outside_the_bf16_tiles_keeps_fp32_probabilities(lib, dh, N):
    Hs, B = 3, 2
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=Hs, d_head=dh, d_ff=8, dtype=BF, max_seq=N)))
    qkv = _dev(_snap(si.normal(dh + N, "qkv", (B * N, 3 * Hs * dh)), BF), BF)
    dout = _dev(_snap(si.normal(N, "dout", (B * N, Hs * dh)), BF), BF)
    o, _, dqkv = ctx.twist_attention_raw(qkv, dout, B, N, Hs)
    torch.cuda.synchronize()
    q, k, v = (to_numpy(qkv).reshape(B, N, 3, Hs, dh)[:, :, i] for i in range(3))
    want_o, p = omodel.attention_fwd(q, k, v)
    want = omodel.attention_bwd(p, q, k, v, to_numpy(dout).reshape(B, N, Hs, dh))
    assert rel_fro(to_numpy(o).reshape(B, N, Hs, dh), want_o) <= 1.8e-3
    for i in range(3):
        assert rel_fro(to_numpy(dqkv).reshape(B, N, 3, Hs, dh)[:, :, i], want[i]) <= 1.8e-3, i


# the 64-row workgroups with fp32 probabilities: lengths around their tiles, one to four of them; rounding of the results as above, the
# log-sum-exp (below 10) within a dozen fp32 roundings; a masked head writes zeros and changes nothing for the others
@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("N", [63, 66, 97, 191, 193, 255])
def test_attention_in_64_row_workgroups(lib, dh, N):
    Hs, B = 3, 2
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=Hs, d_head=dh, d_ff=8, dtype=BF, max_seq=N)))
    qkv = _dev(_snap(si.normal(dh + N, "qkv", (B * N, 3 * Hs * dh)), BF), BF)
    dout = _dev(_snap(si.normal(N, "dout", (B * N, Hs * dh)), BF), BF)
    o, lse, dqkv = ctx.twist_attention_raw(qkv, dout, B, N, Hs)
    om, _, dm = ctx.twist_attention_raw(qkv, dout, B, N, Hs, keep=torch.tensor([4, -1, 0], dtype=torch.int32).cuda())
    torch.cuda.synchronize()
    q, k, v = (to_numpy(qkv).reshape(B, N, 3, Hs, dh)[:, :, i] for i in range(3))
    want_o, p = omodel.attention_fwd(q, k, v)
    want = omodel.attention_bwd(p, q, k, v, to_numpy(dout).reshape(B, N, Hs, dh))
    s = np.einsum("bqhd,bkhd->bhqk", q, k) / np.sqrt(dh)
    s = np.where(np.tril(np.ones((N, N), bool)), s, -np.inf)
    assert np.abs(to_numpy(lse).reshape(B, Hs, N) - np.logaddexp.reduce(s, axis=-1)).max() <= 1e-5
    o, d = to_numpy(o).reshape(B, N, Hs, dh), to_numpy(dqkv).reshape(B, N, 3, Hs, dh)
    om, dm = to_numpy(om).reshape(B, N, Hs, dh), to_numpy(dm).reshape(B, N, 3, Hs, dh)
    assert rel_fro(o, want_o) <= 1.8e-3
    for i in range(3):
        assert rel_fro(d[:, :, i], want[i]) <= 1.8e-3, i
    assert not om[:, :, 1].any() and not dm[:, :, :, 1].any()
    assert np.array_equal(om[:, :, ::2], o[:, :, ::2]) and np.array_equal(dm[:, :, :, ::2], d[:, :, :, ::2])
    for j in (0, N // 2, N - 1):                      # a token whose value row is infinite: earlier queries keep their bits, later ones see it
        x = qkv.clone()
        x.view(B, N, 3, Hs, dh)[0, j, 2, 0, 1] = float("inf")
        oi = to_numpy(ctx.twist_attention_raw(x, None, B, N, Hs)[0]).reshape(B, N, Hs, dh)
        assert np.array_equal(oi[0, :j], o[0, :j]) and np.array_equal(oi[1], o[1]), j
        assert not np.isfinite(oi[0, j, 0, 1]) and np.isfinite(oi[0, :, 0, 2:]).all(), j


# more 128-row workgroups than CUs (3 to 1 blocks of a sequence times many heads): the kernels of 128 rows; the same heads one sequence at a time
# are few enough for the 64-row ones.  Both against the checker, with a head mask, through the rotary backward
@pytest.mark.parametrize("dh,N,Hs,B", [(64, 128, 129, 2), (128, 384, 43, 2), (64, 640, 26, 2)])
def test_attention_with_many_and_with_few_workgroups(lib, dh, N, Hs, B):
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(arch="llama", d_model=64, n_heads=Hs, d_head=dh, d_ff=8, rope=True, dtype=BF, max_seq=N)))
    qkv = _dev(_snap(si.normal(dh + N, "qkv", (B * N, 3 * Hs * dh)), BF), BF)
    dout = _dev(_snap(si.normal(N, "dout", (B * N, Hs * dh)), BF), BF)
    keep_np = np.where(np.arange(Hs) % 5 == 1, -1, 2).astype(np.int32)
    keep, on = torch.tensor(keep_np).cuda(), keep_np >= 0
    many = ctx.twist_attention_raw(qkv, dout, B, N, Hs, keep=keep, rope_backward=True)
    few = ctx.twist_attention_raw(qkv[:N], dout[:N], 1, N, Hs, keep=keep, rope_backward=True)
    torch.cuda.synchronize()
    q, k, v = (to_numpy(qkv[:N]).reshape(1, N, 3, Hs, dh)[:, :, i] for i in range(3))
    want_o, p = omodel.attention_fwd(q, k, v)
    dq, dk, dv = omodel.attention_bwd(p, q, k, v, to_numpy(dout[:N]).reshape(1, N, Hs, dh))
    cos, sin = omodel.rope_tables(N, dh, 1e4)
    want = (omodel.rope_apply(dq, cos, sin, -1.0), omodel.rope_apply(dk, cos, sin, -1.0), dv)
    for o, _, d in (many, few):
        o, d = to_numpy(o[:N]).reshape(1, N, Hs, dh), to_numpy(d[:N]).reshape(1, N, 3, Hs, dh)
        assert not o[:, :, ~on].any() and not d[:, :, :, ~on].any()
        assert rel_fro(o[:, :, on], want_o[:, :, on]) <= 5e-3
        for i in range(3):
            assert rel_fro(d[:, :, i][:, :, on], want[i][:, :, on]) <= 5e-3, i


def test_staged_attention_of_64_wide_heads(lib):
    """The register-staged kernels still serve 64-wide heads of batch elements beyond the pipelined kernels' 2 GiB range."""
    Hs, B, N, dh = 2, 2, 256, 64
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=Hs, d_head=dh, d_ff=8, dtype=BF, max_seq=N)))
    qkv = _dev(_snap(si.normal(3, "qkv", (B * N, 3 * Hs * dh)), BF), BF)
    dout = _dev(_snap(si.normal(4, "dout", (B * N, Hs * dh)), BF), BF)
    a = ctx.twist_attention_raw(qkv, dout, B, N, Hs)
    ctx.twist_set_kernel_choice(staged_attention=True)
    b = ctx.twist_attention_raw(qkv, dout, B, N, Hs)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert rel_fro(to_numpy(x), to_numpy(y)) <= 5e-3


# fp32: head widths below, at and above a 32-column block; lengths below, at and beyond a 32-row tile and beyond four of them
@pytest.mark.parametrize("dh", [4, 16, 32, 36, 64, 128])
@pytest.mark.parametrize("N", [1, 31, 32, 33, 97, 160, 200])
def test_fp32_attention_of_any_length(lib, dh, N):
    Hs, B = 3, 2
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=Hs, d_head=dh, d_ff=8, max_seq=N)))
    qkv = _dev(_snap(si.normal(dh + N, "qkv", (B * N, 3 * Hs * dh)), F32), F32)
    dout = _dev(_snap(si.normal(N, "dout", (B * N, Hs * dh)), F32), F32)
    q, k, v = (to_numpy(qkv).reshape(B, N, 3, Hs, dh)[:, :, i] for i in range(3))
    g = to_numpy(dout).reshape(B, N, Hs, dh)
    want_o, p = omodel.attention_fwd(q, k, v)
    want = omodel.attention_bwd(p, q, k, v, g)
    for keep_np in (None, np.array([0, -1, 3], np.int32)):
        on = np.ones(Hs, bool) if keep_np is None else keep_np >= 0
        o, lse, dqkv = ctx.twist_attention_raw(qkv, dout, B, N, Hs, keep=None if keep_np is None else torch.tensor(keep_np).cuda())
        torch.cuda.synchronize()
        o, got = to_numpy(o).reshape(B, N, Hs, dh), to_numpy(dqkv).reshape(B, N, 3, Hs, dh)
        assert rel_fro(o[:, :, on], want_o[:, :, on]) <= 3e-6
        assert not o[:, :, ~on].any() and not got[:, :, :, ~on].any()
        for i in range(3):
            # a sequence of one has dq = dk = 0 in exact arithmetic; what is left is the rounding of dp - delta, 1e-7 of |dO| |v| |k|
            err = np.linalg.norm(got[:, :, i][:, :, on] - want[i][:, :, on])
            assert err <= 1e-5 * np.linalg.norm(want[i][:, :, on]) + 1e-6 * np.linalg.norm(g) * dh, (i, err)


# fp32: more tiles of 32 than four waves, in few workgroups (eight waves each) and many (four): the same sequences give the same results
@pytest.mark.parametrize("dh", [32, 36, 64])
@pytest.mark.parametrize("N", [129, 160, 289])
def test_fp32_attention_of_few_and_many_workgroups(lib, dh, N):
    Hs, many = 3, 40
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=Hs, d_head=dh, d_ff=8, max_seq=N)))
    assert (N + 31) // 32 * Hs <= 512 < (N + 31) // 32 * Hs * many
    qkv = _dev(_snap(si.normal(dh + N, "qkv", (N, 3 * Hs * dh)), F32), F32)
    dout = _dev(_snap(si.normal(N, "dout", (N, Hs * dh)), F32), F32)
    few = ctx.twist_attention_raw(qkv, dout, 1, N, Hs)
    more = ctx.twist_attention_raw(qkv.repeat(many, 1), dout.repeat(many, 1), many, N, Hs)
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(few, more)):
        b = b.view(many, *a.shape)
        assert torch.equal(b, b[:1].expand_as(b))
        # both as far from exact arithmetic as the oracle comparison above allows, 3e-6 forward and 1e-5 backward
        assert rel_fro(to_numpy(b[0]), to_numpy(a)) <= (6e-6 if i < 2 else 2e-5), i


# ... and sequences of a few tiles more than four waves have four to a workgroup as soon as there are more workgroups than CUs: the bits of the same ones among many
@pytest.mark.parametrize("dh", [32, 64])
@pytest.mark.parametrize("N,B", [(129, 18), (160, 18), (256, 11), (257, 15), (320, 13)])
def test_fp32_attention_of_short_sequences_on_full_cus(lib, dh, N, B):
    Hs, many = 3, 40
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=Hs, d_head=dh, d_ff=8, max_seq=N)))
    assert (256 if N <= 256 else 384) < (N + 31) // 32 * Hs * B <= 512 < (N + 31) // 32 * Hs * many
    qkv = _dev(_snap(si.normal(dh + N, "qkv", (N, 3 * Hs * dh)), F32), F32)
    dout = _dev(_snap(si.normal(N, "dout", (N, Hs * dh)), F32), F32)
    some, more = (ctx.twist_attention_raw(qkv.repeat(n, 1), dout.repeat(n, 1), n, N, Hs) for n in (B, many))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b[:len(a)]) for a, b in zip(some, more))


# An infinity or a NaN in one token's value, key, query or output gradient: what does not depend on it keeps its bits (earlier queries'
# outputs and gradients; for a query or an output gradient, later keys' too), and what the plain kernels, which visit visible pairs only,
# compute as finite is finite.  Tokens inside a 32-row tile, at its edges and last of a ragged one.  (bf16 at 128 and 256 tokens: the 64-row workgroups with
# probabilities rounded to bf16.)
@pytest.mark.parametrize("dtype,dh,N", [(F32, 36, 70), (F32, 64, 70), (F32, 128, 70), (BF, 32, 70), (BF, 128, 70), (BF, 64, 128), (BF, 128, 128), (BF, 64, 256)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_attention_keeps_a_non_finite_token_from_what_does_not_see_it(lib, dtype, dh, N, value):
    Hs, B = 2, 2
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=Hs, d_head=dh, d_ff=8, dtype=dtype, max_seq=N)))
    qkv = _dev(_snap(si.normal(dh, "qkv", (B * N, 3 * Hs * dh)), dtype), dtype)
    dout = _dev(_snap(si.normal(N, "dout", (B * N, Hs * dh)), dtype), dtype)

    def run(x, g):
        o, _, d = ctx.twist_attention_raw(x, g, B, N, Hs)
        return [t.view(B, N, Hs, dh) for t in (o, *d.view(B, N, 3, Hs, dh).unbind(2))]

    clean = run(qkv, dout)
    for what in range(4):          # query, key, value, output gradient
        for j in (5, 32, 47, 63, 69, N - 1):
            x, g = qkv.clone(), dout.clone()
            if what < 3:
                x.view(B, N, 3, Hs, dh)[0, j, what, 1, 3] = value
            else:
                g.view(B, N, Hs, dh)[0, j, 1, 3] = value
            got = run(x, g)
            ctx.twist_set_kernel_choice(plain_only=True)
            plain = run(x, g)
            ctx.twist_set_kernel_choice()
            torch.cuda.synchronize()
            for i, (a, b, c) in enumerate(zip(got, plain, clean)):
                assert torch.equal(a[1], c[1]) and torch.equal(a[:, :, 0], c[:, :, 0]), (what, j, i)      # the other sequence, the other head
                if i < 2:
                    assert torch.equal(a[0, :j], c[0, :j]), (what, j, i)
                elif what in (0, 3):
                    assert torch.equal(a[0, j + 1:], c[0, j + 1:]), (what, j, i)
                assert bool((torch.isfinite(a) | ~torch.isfinite(b)).all()), (what, j, i)
            # and where it belongs it shows: in the token's own output, or its query's gradient (an infinite key may have weight zero)
            if what != 1 or value != value:
                assert not torch.isfinite(got[0 if what < 3 else 1][0, j, 1]).all(), (what, j)


# fp32 attention keeps the precision of the plain kernels, which visit one key at a time and add pairwise: error against the fp64 checker
# at most 1.35 times theirs (both are a few roundings of 2^-24; the order of sums alone moves it by up to 1.2), on plain normal operands,
# on scores of about +-30 (what is rounded there must be score differences, not scores) and with a component common to all value rows
@pytest.mark.parametrize("dh,N", [(32, 64), (64, 320), (128, 200)])
@pytest.mark.parametrize("kind", ["normal", "sharp", "bias", "both"])
def test_fp32_attention_is_as_precise_as_the_plain_kernels(lib, dh, N, kind):
    Hs, B = 3, 2
    ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=Hs, d_head=dh, d_ff=8, max_seq=N)))
    x = si.normal(dh + N, "qkv", (B * N, 3, Hs * dh))
    if kind in ("sharp", "both"):
        x[:, 0] *= 8
    if kind in ("bias", "both"):
        x[:, 2] += 20
    qkv = _dev(_snap(x.reshape(B * N, -1), F32), F32)
    dout = _dev(_snap(si.normal(N, "dout", (B * N, Hs * dh)), F32), F32)
    q, k, v = (to_numpy(qkv).reshape(B, N, 3, Hs, dh)[:, :, i] for i in range(3))
    want_o, p = omodel.attention_fwd(q, k, v)
    want = (want_o, *omodel.attention_bwd(p, q, k, v, to_numpy(dout).reshape(B, N, Hs, dh)))
    err = []
    for plain in (False, True):
        ctx.twist_set_kernel_choice(plain_only=plain)
        o, _, d = ctx.twist_attention_raw(qkv, dout, B, N, Hs)
        torch.cuda.synchronize()
        got = (to_numpy(o).reshape(B, N, Hs, dh), *np.moveaxis(to_numpy(d).reshape(B, N, 3, Hs, dh), 2, 0))
        err.append([rel_fro(a, b) for a, b in zip(got, want)])
    assert all(a <= 1.35 * b for a, b in zip(*err)), err


def test_cross_entropy_leaves_out_what_lies_beyond_a_short_row(lib):
    """Rows of 515 and of 4096 logits run the same kernel, which has room for 8192: an eighth of the row is at most 0.8 of the time
    (measured 0.65; 0.92 where every lane works on all of its four vectors)."""
    us = []
    for V in (515, 4096):
        ctx = lib.Context(lib.desc_from_cfg(si.ModelCfg(d_model=64, n_heads=1, d_head=8, d_ff=8, vocab=V, dtype=BF)))
        logits = torch.randn(32768, (V + 7) // 8 * 8, device="cuda").bfloat16()
        y = torch.randint(0, V, (32768,), device="cuda", dtype=torch.int32)
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                ctx.twist_ce_raw(logits, y)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) / 4 * 1e3)
        us.append(min(times))
    assert us[0] <= 0.8 * us[1], us
