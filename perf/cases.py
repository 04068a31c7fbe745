"""The work that a user has this library do, as cases that can be timed: whole rounds, training steps, gradients, evaluation,
the masked variant and the traffic between two rounds, each through the entry points of the binding.

A case is a dict of plain values: the model (`arch`, `layers`, `d`, `heads`, `dh`, `ff`, `granule`, `vocab`, `dtype`, `um` = output
projections stored unit-major), the blueprint (`S` subnets of `hs` heads and `fs` blocks of `granule` neurons, the first and last
`shared` layers kept whole), the batch (`B` sequences of `N` tokens, ids uniform or, with `zipf`, Zipf(1.1)) and what is done with
them (`kind`):

  round    twist_round on a persistent central model: sample, then extract, train `steps` batches and add to the running
           average for each subnet, finally write the averages back
  train    one local step of one subnet: twist_subnet_fwd_bwd, then twist_subnet_step with AdamW
  grads    twist_subnet_fwd_bwd alone
  masked   twist_subnet_fwd_bwd_masked: the full-width model under one blueprint row's mask
  forward  twist_subnet_forward: evaluation of a deployed subnet
  move     what happens between two rounds when all subnets are resident: twist_aggregate of the trained subnets, twist_sample
           of the next blueprint, twist_extract_all into the next round's storage
"""
from __future__ import annotations

import math

import torch

import paper_2511_03983_amd as tw
from synth_inputs import ModelCfg, global_shapes, stored_shapes

GPT2S = {"arch": "gpt", "layers": 12, "d": 768, "heads": 12, "dh": 64, "ff": 3072, "vocab": 50257}
LLAMA1B = {"arch": "llama", "d": 2048, "heads": 16, "dh": 128, "ff": 5632, "vocab": 32000}
LLAMA7B = {"arch": "llama", "d": 4096, "heads": 32, "dh": 128, "ff": 11008}


def _case(kind, model, dtype="bf16", um=True, granule=1, shared=0, S=1, steps=1, zipf=False, **more):
    return {"kind": kind, **model, "dtype": dtype, "um": um, "granule": granule, "shared": shared, "S": S, "steps": steps, "zipf": zipf, **more}


def listed():
    """Sizes are those of the repository's workloads and tests; the Llama-shaped 7B stacks are cut to a few of their 32
    identical layers so that a state fits the card several times, and the masked and ragged ones likewise."""
    return [
        # smallest: a whole round of the tiny fp32 block (smoke, unit tests, the train-X / eval-Y grid's scale): latency and launches
        {"name": "round_block_f32", **_case("round", {"arch": "gpt", "layers": 1, "d": 128, "heads": 4, "dh": 32, "ff": 512, "vocab": 0}, "f32", False,
                                            S=2, hs=2, fs=256, B=4, N=64)},
        # a round as it is trained at GPT-2-small shape, one subnet resident at a time, two local AdamW batches each
        {"name": "round_gpt_small", **_case("round", GPT2S, S=4, hs=3, fs=768, B=8, N=1024, steps=2)},
        # the same model kept in fp32 throughout, one local step of a half-width subnet
        {"name": "train_gpt_f32", **_case("train", GPT2S, "f32", False, S=2, hs=6, fs=1536, B=2, N=512)},
        # latency study of the paper: 8 of 12 blocks kept, first and last two layers shared, [out, in] storage, 2 x 1024 tokens
        {"name": "train_gpt_blocks", **_case("train", GPT2S, um=False, granule=256, shared=2, S=3, hs=8, fs=8, B=2, N=1024)},
        # four disjoint quarter-width subnets, the workload's batch: narrow matrices, a vocabulary projection that outweighs them
        {"name": "grads_gpt_quarter", **_case("grads", GPT2S, S=4, hs=3, fs=768, B=8, N=1024)},
        # deployment: a pruned model answering one short and one full-length request
        {"name": "forward_gpt_short", **_case("forward", GPT2S, um=False, granule=256, shared=2, hs=6, fs=6, B=1, N=128)},
        {"name": "forward_gpt_full", **_case("forward", GPT2S, um=False, granule=256, shared=2, hs=10, fs=10, B=4, N=1024)},
        # the benchmark's local step: half-width Llama-shaped 1B subnet, 4 x 2048 Zipf tokens, AdamW (the largest)
        {"name": "train_llama1b_half", **_case("train", LLAMA1B, layers=22, S=4, hs=8, fs=2816, B=4, N=2048, zipf=True)},
        # sequences and widths as data give them: nothing a multiple of a tile
        {"name": "grads_llama_ragged", **_case("grads", LLAMA1B, um=False, granule=8, layers=6, S=3, hs=7, fs=311, B=3, N=1000)},
        # Masked TwIST: the full-width model under a half-width mask
        {"name": "masked_llama1b", **_case("masked", LLAMA1B, layers=6, S=4, hs=8, fs=2816, B=4, N=2048)},
        # pruned-once 7B widths, long sequences
        {"name": "grads_llama7b_pruned", **_case("grads", {**LLAMA7B, "vocab": 32000}, layers=4, hs=16, fs=5504, B=2, N=4096)},
        # aggregate, resample, dispatch at 7B widths, neuron blocks as rows and as columns of the down projection
        {"name": "move_llama7b_rows", **_case("move", {**LLAMA7B, "vocab": 0}, layers=8, S=8, hs=16, fs=5504, B=1, N=1)},
    ]


def draw(rng):
    """One more case: any kind, sizes spread over the ranges above, half of the sequence lengths and widths with no factor in common
    with a tile; never more work than the benchmark's local step."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    while True:
        kind = rng.choice(["round", "train", "grads", "grads", "forward", "masked", "move"])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        um = rng.random() < 0.5
        if rng.random() < 0.5:
            dh = rng.choice([32, 64, 64, 64])
            heads = rng.randint(2, 16)
            d = log(64, 1024) // 8 * 8
            m = {"arch": "gpt", "d": d, "heads": heads, "dh": dh, "ff": 4 * d, "layers": rng.randint(1, 12)}
        else:
            dh = rng.choice([64, 128, 128, 128])
            d = log(256, 4096) // 8 * 8
            heads = max(2, d // dh)
            m = {"arch": "llama", "d": d, "heads": heads, "dh": dh, "ff": int(2.75 * d) // 8 * 8, "layers": rng.randint(1, 8 if d > 2048 else 22)}
        granule = rng.choice([1, 8, m["ff"] // 8 if m["ff"] % 64 == 0 else 8])   # kept widths are multiples of 8
        units = m["ff"] // granule
        S = rng.randint(1, 8) if kind in ("round", "move") else rng.randint(1, 4)
        keep = rng.uniform(0.25, 1.0)
        hs = min(heads, max(-(-heads // S), int(round(keep * heads))))
        fs = min(units, max(-(-units // S), int(round(keep * units))))
        if granule == 1:
            fs = min(units, -(-fs // 8) * 8)
        m["vocab"] = 0 if kind == "move" else rng.choice([0, 1003, 32000, 50257])
        N = log(33, 4096)
        if rng.random() < 0.5:
            N = max(64, N // 64 * 64)
        B = rng.randint(1, 8)
        if B * N > 8192:
            continue
        c = _case(kind, m, dtype, um, granule, rng.choice([0, 0, 1]) if m["layers"] > 2 else 0, S, hs=hs, fs=fs, B=B if kind != "move" else 1,
                  N=N if kind != "move" else 1, zipf=rng.random() < 0.3)
        w = work(c)
        pairs = c["S"] ** (kind == "round") * B * heads * m["layers"] * N * N
        if kind == "move" and not 1e6 < w["bytes"] < 2.6e10:
            continue
        if w["flops"] > (1.5e13 if dtype == "bf16" else 8e11) or pairs > 2e9 or (kind != "move" and w["bytes"] > 2e10):
            continue
        return c


# ---------------------------------------------------------------------------------------------- sizes
def _cfg(c):
    llama = c["arch"] == "llama"
    return ModelCfg(arch=c["arch"], n_layers=c["layers"], d_model=c["d"], n_heads=c["heads"], d_head=c["dh"], d_ff=c["ff"], ffn_granule=c["granule"],
                    vocab=c["vocab"], max_seq=c["N"], act="swiglu" if llama else "gelu_tanh", norm="rms" if llama else "ln", has_bias=not llama,
                    tied_head=not llama, rope=llama, dtype=c["dtype"], out_unit_major=c["um"])


def _layer_shared(c):
    n = c["shared"]
    return [1] * n + [0] * (c["layers"] - 2 * n) + [1] * n if n else None


def _params(c):
    """(partitioned-and-kept + shared parameters of one subnet, parameters of the central model)"""
    cfg = _cfg(c)
    full = kept = 0
    for l in range(c["layers"]):
        whole = c["shared"] and (l < c["shared"] or l >= c["layers"] - c["shared"])
        for k, s in stored_shapes(cfg).items():
            n = math.prod(s)
            head = k in ("wq", "wk", "wv", "wo", "bq", "bk", "bv")
            ffn = k in ("w_gate", "w_up", "w_down", "b_up")
            full += n
            kept += n if whole or not (head or ffn) else n * c["hs"] // c["heads"] if head else n * c["fs"] // (c["ff"] // c["granule"])
    g = sum(math.prod(s) for s in global_shapes(cfg).values())
    return kept + g, full + g


def work(c):
    """Projections 2 M N K, causal attention at half of 4 B H N^2 d_head, backward twice the forward; every parameter, gradient and
    optimizer value once per use."""
    es = 2 if c["dtype"] == "bf16" else 4
    kept, full = _params(c)
    if c["kind"] == "move":   # aggregate: subnets read, central written; dispatch: central read, subnets written
        return {"bytes": es * 2 * (c["S"] * kept + full), "flops": 0}
    T, nf = c["B"] * c["N"], 2 if c["arch"] == "llama" else 1
    fwd = 0.0
    for l in range(c["layers"]):
        whole = c["shared"] and (l < c["shared"] or l >= c["layers"] - c["shared"])
        h = c["heads"] if whole else c["hs"]
        f = c["ff"] if whole else c["fs"] * c["granule"]
        fwd += 2 * T * c["d"] * (4 * h * c["dh"] + (nf + 1) * f) + 2 * c["B"] * h * c["N"] ** 2 * c["dh"]
    fwd += 2 * T * c["d"] * c["vocab"]
    io = T * (8 if c["vocab"] else 2 * es * c["d"])
    if c["kind"] == "forward":
        return {"bytes": es * kept + io, "flops": fwd}
    grads = es * kept + 4 * kept + io
    step = (4 + 8 + 16 + (es if es == 2 else 0)) * kept           # AdamW: gradient, master, two moments, the bf16 copy
    if c["kind"] == "grads":
        return {"bytes": grads, "flops": 3 * fwd}
    if c["kind"] == "masked":
        return {"bytes": es * kept + 4 * full + io, "flops": 3 * fwd}
    if c["kind"] == "train":
        return {"bytes": grads + step, "flops": 3 * fwd}
    return {"bytes": c["S"] * (c["steps"] * (grads + step) + 2 * es * kept) + es * full, "flops": 3 * fwd * c["S"] * c["steps"]}


def tolerance(c):
    """About four times what the library's kernel families (tile sizes, fp32-arithmetic kernels) differ by on the listed cases: up to
    6e-3 between tile sizes, 1.3e-2 against fp32 arithmetic (loss alone 4e-5), single entries up to 0.6 of the rms (the frequent rows of
    an embedding gradient are many times that rms, and so are their errors).  fp32: four times the distance from the fp64 checker
    (3e-6); there AdamW's first step moves a weight by its learning rate whatever the size of its gradient, so a gradient whose sign is
    noise moves it by 2e-4 where the weights' rms is 0.02: `max` 0.01."""
    if c["kind"] == "move":
        return "exact"           # copies, and fp32 sums in the order given, rounded once
    if c["dtype"] == "f32":
        return {"rel": 2e-5, "max": 0.04 if c["kind"] in ("train", "round") and c["vocab"] else 2e-3}
    return {"rel": 2e-4} if c["kind"] == "forward" else {"rel": 2.5e-2, "max": 0.99}


# ---------------------------------------------------------------------------------------------- inputs
def _normal(n, dtype, gen, std):
    out = torch.empty(n, dtype=dtype, device="cuda")
    step = 1 << 26
    for o in range(0, n, step):
        k = min(step, n - o)
        out[o:o + k] = torch.randn(k, generator=gen, device="cuda") * std
    return out


def _central(cfg, gen):
    """The central model in one flat buffer: N(0, 0.02) matrices and biases, gains near 1; and its tensors by name."""
    dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    up = lambda n: (n + 127) // 128 * 128  # noqa: E731
    shapes = [stored_shapes(cfg)] * cfg.n_layers + [global_shapes(cfg)]
    flat = _normal(sum(up(math.prod(s)) for t in shapes for s in t.values()), dt, gen, 0.02)
    off, named = 0, []
    for t in shapes:
        views = {}
        for k, s in t.items():
            v = flat[off:off + math.prod(s)].view(s)
            if len(s) == 1 and k.endswith("_w"):
                v += 1
            views[k] = v
            off += up(math.prod(s))
        named.append(views)
    return flat, tw.FullWeights(named[:-1], named[-1])


def _batch(c, cfg, lead, gen):
    """Inputs and targets of shape lead + (B, N): token ids and the same shifted by one, or N(0, 1) activations."""
    shape = lead + (c["B"], c["N"])
    if not cfg.vocab:
        dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
        return tuple(torch.randn(shape + (cfg.d_model,), generator=gen, device="cuda").to(dt) for _ in range(2))
    u = torch.rand(lead + (c["B"], c["N"] + 1), generator=gen, device="cuda", dtype=torch.float64)
    if c["zipf"]:
        cdf = torch.arange(1, cfg.vocab + 1, device="cuda", dtype=torch.float64).pow_(-1.1).cumsum_(0)
        t = torch.searchsorted(cdf, u * cdf[-1])
    else:
        t = (u * cfg.vocab).floor()
    t = t.clamp_(max=cfg.vocab - 1).to(torch.int32)
    return t[..., :-1].contiguous(), t[..., 1:].contiguous()


def _regions(sub, cfg, what):
    """A subnet's storage region as three tensors: the layers' matrices, the model-level matrices, the vectors."""
    first = sub.twist_subnet_view(0, "wq", what)
    glob = sub.twist_subnet_view(-1, "tok_embed", what) if cfg.vocab else None
    vec = sub.twist_subnet_view(0, "bq" if cfg.has_bias else "norm1_w", what)
    es = first.element_size()
    a = first.data_ptr() - sub.storage.data_ptr()
    v = vec.data_ptr() - sub.storage.data_ptr()
    g = glob.data_ptr() - sub.storage.data_ptr() if cfg.vocab else v
    last = sub.twist_subnet_view(-1, "final_norm_b" if cfg.norm == "ln" else "final_norm_w", what) if cfg.vocab else \
        sub.twist_subnet_view(cfg.n_layers - 1, "norm2_b" if cfg.norm == "ln" else "norm2_w", what)
    end = last.data_ptr() - sub.storage.data_ptr() + last.numel() * es
    cut = lambda lo, hi: sub.storage[lo:hi].view(first.dtype)  # noqa: E731
    return [cut(a, g), cut(g, v), cut(v, end)] if cfg.vocab else [cut(a, v), cut(v, end)]


class State:
    pass


def prepare(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    cfg, s = _cfg(c), State()
    s.case, s.cfg = c, cfg
    flat, full = _central(cfg, gen)
    s.ctx = tw.Context(tw.desc_from_cfg(cfg))
    s.blueprint = dict(S=c["S"], heads_sub=c["hs"], ffn_units_sub=c["fs"], layer_shared=_layer_shared(c))
    cover = c["S"] * c["hs"] >= c["heads"] and c["S"] * c["fs"] >= c["ff"] // c["granule"]
    s.seed = seed % 1000
    room = lambda n: torch.zeros(n, dtype=torch.uint8, device="cuda")  # noqa: E731
    if c["kind"] == "move":
        s.flat, s.full = flat, full
        s.plan = s.ctx.twist_sample(**s.blueprint, seed=s.seed, rnd=0, require_coverage=cover)
        nb = s.ctx.twist_subnet_bytes(s.plan)
        s.subs = s.ctx.twist_extract_all(s.plan, full, storages=[room(nb) for _ in range(c["S"])])
        dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
        for sub in s.subs:   # stands for the local training
            w = sub.storage.view(dt)
            w += _normal(w.numel(), dt, gen, 1e-3)
        s.next = [room(nb) for _ in range(c["S"])]
        s.cover = cover
        return s
    if c["kind"] == "round":
        s.flat, s.full = flat, full
        s.x, s.y = _batch(c, cfg, (c["S"], c["steps"]), gen)
        s.opt = {"kind": tw.OPT_SGD, "lr": 1e-2} if not cfg.vocab else {"kind": tw.OPT_ADAMW, "lr": 1e-4, "weight_decay": 0.01}
        sb, wb, ib = s.ctx.twist_round_bytes(c["S"], c["hs"], c["fs"], c["B"], c["N"], c["steps"], opt=s.opt, layer_shared=_layer_shared(c))
        s.slab, s.ws, s.image = room(sb), torch.empty(wb, dtype=torch.uint8, device="cuda"), torch.empty(ib, dtype=torch.uint8, device="cuda")
        s.loss = torch.zeros(c["S"], c["steps"], device="cuda")
        return s
    s.plan = s.ctx.twist_sample(**s.blueprint, seed=s.seed, require_coverage=cover)
    source = s.plan
    if c["kind"] == "masked":
        source = s.whole = s.ctx.twist_sample(1, c["heads"], c["ff"] // c["granule"], seed=s.seed)
    store = {"forward": tw.STORE_PARAMS, "train": tw.STORE_ADAMW}.get(c["kind"], tw.STORE_GRADS)
    s.sub = s.ctx.twist_extract(source, full, 0, store=store, storage=room(s.ctx.twist_subnet_bytes(source, store)))
    s.x, s.y = _batch(c, cfg, (), gen)
    s.ws = torch.empty(s.ctx.twist_workspace_bytes(s.sub, c["B"], c["N"]), dtype=torch.uint8, device="cuda")
    s.loss = torch.zeros(1, device="cuda")
    return s


def run(s):
    c, ctx = s.case, s.ctx
    kind = c["kind"]
    if kind == "move":
        ctx.twist_aggregate(s.plan, s.subs, s.full)
        plan = ctx.twist_sample(**s.blueprint, seed=s.seed, rnd=1, require_coverage=s.cover)
        for sub in ctx.twist_extract_all(plan, s.full, storages=s.next):
            sub.close()
        plan.close()
        return {"central": s.flat, "subnets": s.next}
    if kind == "round":
        ctx.twist_round(s.full, s.x, s.y, c["S"], c["hs"], c["fs"], s.slab, s.ws, s.image, s.loss, seed=s.seed, opt=s.opt, layer_shared=_layer_shared(c))
        return {"loss": s.loss, "central": s.flat}
    if kind == "forward":
        ctx.twist_subnet_forward(s.sub, s.x, s.y, s.ws, s.loss)
        return {"loss": s.loss}
    if kind == "masked":
        ctx.twist_subnet_fwd_bwd_masked(s.sub, s.plan, 0, s.x, s.y, s.ws, s.loss)
    else:
        ctx.twist_subnet_fwd_bwd(s.sub, s.x, s.y, s.ws, s.loss)
    out = {"loss": s.loss}
    if kind == "train":
        ctx.twist_subnet_step(s.sub, tw.OPT_ADAMW, lr=1e-4, weight_decay=0.01)
        for name, what in (("weights", tw.binding.PARAM), ("master", tw.binding.MASTER), ("moment1", tw.binding.ADAM_M), ("moment2", tw.binding.ADAM_V)):
            out[name] = _regions(s.sub, s.cfg, what)
    out["grads"] = _regions(s.sub, s.cfg, tw.binding.GRAD)
    return out
