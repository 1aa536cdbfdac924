"""The workloads this library's speed is judged on: what a training program asks of it, through the public entry points.

A case is one of nine kinds of work (`kind`), each a forward and the backward that belongs to it, or one optimizer step:

  layer      the non-GEMM calls of one pre-LayerNorm encoder layer, forward and backward (12 calls; 17 with padding removed)
  sublayer   the boundary of a sub-layer: bias + dropout + residual and the LayerNorm behind it, fused or as four calls
  softmax    masked attention softmax, forward and backward
  ffn        bias + activation + dropout of the feed-forward block, forward and backward
  heads      the "Reshape" calls of an attention block: QKV split and head merge, forward and backward
  embedding  token + position embedding and the accumulation of its gradient
  criterion  label-smoothed cross-entropy over the vocabulary, as one pass or as two calls
  trainer    one optimizer step over a flat workspace
  padding    length offsets, padding removal and its inverse

`graph` says that the program has captured the calls into a HIP graph once and replays it, which is what a program whose
kernels are shorter than their launches does; the other cases call the entry points from Python and let them allocate
their outputs.  GEMM results between the calls (projections, scores, upstream gradients) are inputs made beforehand.
"""
from __future__ import annotations

import math

import torch

import paper_2110_05722_amd as L

DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"f16": 2, "bf16": 2, "f32": 4}
IGNORE = -100
PAD = 1
EPS = 1e-5
ADAM = dict(lr=1e-3, beta1=0.9, beta2=0.98, eps=1e-8)
SGD = dict(lr=1e-2, momentum=0.9)
FIRST_STEP = 1000          # the optimizer's step count when the program reaches the measured step
PHILOX_SEED = 1234


# ------------------------------------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest call pattern: a layer of a small model, every call issued from Python
        dict(name="layer-tiny-f32", kind="layer", dt="f32", batch=8, len=64, heads=8, head_dim=64, ffn=2048, act="relu",
             p=0.1, p_attn=0.0, packed=False, graph=False),
        # transformer-base on sentence pairs of uneven length: padding removed, the layer captured as a graph
        dict(name="layer-transformer-base-f16", kind="layer", dt="f16", batch=128, len=32, heads=8, head_dim=64, ffn=2048,
             act="relu", p=0.1, p_attn=0.1, packed=True, graph=True),
        # gpt2-large, the boundary between attention and feed-forward block in one pass
        dict(name="sublayer-gpt2-large-bf16", kind="sublayer", dt="bf16", rows=8192, hidden=1280, p=0.1, fused=True, graph=False),
        # bert-large with the four separate entry points, captured
        dict(name="sublayer-bert-large-f16", kind="sublayer", dt="f16", rows=8192, hidden=1024, p=0.1, fused=False, graph=True),
        # gpt2-large causal self-attention, no attention dropout
        dict(name="softmax-gpt2-large-bf16", kind="softmax", dt="bf16", batch=8, heads=20, q_len=1024, k_len=1024,
             causal=True, ragged=False, p_attn=0.0, graph=False),
        # transformer-big self-attention on a batch padded to its longest sentence, whatever that length is
        dict(name="softmax-ragged-f16", kind="softmax", dt="f16", batch=64, heads=16, q_len=113, k_len=113,
             causal=False, ragged=True, p_attn=0.1, graph=False),
        # bert-large feed-forward block, GELU
        dict(name="ffn-bert-large-bf16", kind="ffn", dt="bf16", rows=8192, hidden=4096, act="gelu", p=0.1, graph=False),
        # gpt2-large QKV split and head merge
        dict(name="heads-gpt2-large-f16", kind="heads", dt="f16", batch=8, len=1024, heads=20, head_dim=64, parts=3, graph=False),
        # gpt2-large embedding on text (a few words make up much of it)
        dict(name="embedding-gpt2-large-bf16", kind="embedding", dt="bf16", batch=8, len=1024, hidden=1280, vocab=50257,
             ragged=False, p=0.1, graph=False),
        # gpt2-large language-model criterion, loss and gradient in one pass
        dict(name="criterion-gpt2-large-f16", kind="criterion", dt="f16", tokens=8192, vocab=50257, alpha=0.1, active=1.0,
             one_pass=True, graph=False),
        # bert-large masked-LM criterion: 15 % of the positions carry a target, forward and backward as two calls
        dict(name="criterion-masked-lm-bf16", kind="criterion", dt="bf16", tokens=8192, vocab=30522, alpha=0.0, active=0.15,
             one_pass=False, graph=False),
        # bert-large mixed-precision Adam
        dict(name="trainer-bert-large-f16", kind="trainer", dt="f16", n=335_000_000, rule="adam", graph=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _hidden(rng, lo, hi):
    """A row length: three in four a multiple of 8 as model widths are, else anything."""
    h = _log(rng, lo, hi)
    return max(8, h - h % 8) if rng.random() < 0.75 else h


def draw(rng):
    kind = rng.choice(["layer", "sublayer", "softmax", "ffn", "heads", "embedding", "criterion", "trainer", "padding"])
    dt = rng.choice(["f16", "f16", "bf16", "bf16", "f32"])
    graph = rng.random() < 0.3
    p = rng.choice([0.0, 0.1, 0.3])
    if kind == "layer":
        ln = rng.randint(16, 256)
        return dict(kind=kind, dt=dt, batch=max(2, min(256, _log(rng, 512, 8192) // ln)), len=ln, heads=rng.randint(4, 20),
                    head_dim=rng.choice([64, 64, 80]), ffn=8 * rng.randint(128, 640), act=rng.choice(["relu", "gelu", "gelu_tanh"]),
                    p=p, p_attn=rng.choice([0.0, 0.1]), packed=rng.random() < 0.5, graph=graph)
    if kind == "sublayer":
        hidden = _hidden(rng, 256, 8192)
        return dict(kind=kind, dt=dt, rows=_log(rng, 500, min(16384, 33_000_000 // hidden)), hidden=hidden, p=p,
                    fused=rng.random() < 0.5, graph=graph)
    if kind == "softmax":
        k_len = _log(rng, 16, 4096)
        q_len = k_len if rng.random() < 0.7 else _log(rng, 16, 2048)
        heads = rng.randint(4, 20)
        most = max(1, min(128, 168_000_000 // (heads * q_len * k_len)))
        return dict(kind=kind, dt=dt, batch=rng.randint(max(1, most // 8), most), heads=heads, q_len=q_len, k_len=k_len,
                    causal=rng.random() < 0.4, ragged=rng.random() < 0.6, p_attn=rng.choice([0.0, 0.1]), graph=graph)
    if kind == "ffn":
        hidden = _hidden(rng, 1024, 16384)
        return dict(kind=kind, dt=dt, rows=_log(rng, 500, min(16384, 67_000_000 // hidden)), hidden=hidden,
                    act=rng.choice(["relu", "gelu", "gelu_tanh"]), p=p, graph=graph)
    if kind == "heads":
        ln = _log(rng, 16, 1024)
        return dict(kind=kind, dt=dt, batch=max(1, _log(rng, 512, 16384) // ln), len=ln, heads=rng.randint(4, 20),
                    head_dim=rng.choice([32, 64, 64, 80, 128]), parts=rng.choice([1, 2, 3, 3]), graph=graph)
    if kind == "embedding":
        ln = _log(rng, 16, 1024)
        hidden = _hidden(rng, 256, 2048)
        return dict(kind=kind, dt=dt, batch=max(1, _log(rng, 512, 20000) // ln), len=ln, hidden=hidden,
                    vocab=_log(rng, 8000, 65536), ragged=rng.random() < 0.5, p=p, graph=graph)
    if kind == "criterion":
        vocab = _log(rng, 8000, 131072)
        return dict(kind=kind, dt=dt, tokens=_log(rng, 300, 411_000_000 // vocab), vocab=vocab, alpha=rng.choice([0.0, 0.1]),
                    active=rng.choice([0.15, 0.5, 0.8, 1.0]), one_pass=rng.random() < 0.5, graph=graph)
    if kind == "trainer":
        return dict(kind=kind, dt=dt if dt != "f32" else "f16", n=_log(rng, 1_000_000, 335_000_000),
                    rule=rng.choice(["adam", "adam_blocked", "adam_lp", "sgd", "sgd_blocked"]), graph=False)
    ln = _log(rng, 16, 1024)
    return dict(kind=kind, dt=dt, batch=max(2, _log(rng, 512, 16384) // ln), len=ln, hidden=_hidden(rng, 256, 4096), graph=graph)


# ------------------------------------------------------------------------------------------------------ inputs
def _lengths(case, gen):
    """int32[batch] sentence lengths on the GPU: log-normal about half the padded length (sigma 0.5), one sentence full.
    The mix belongs to the case (sum known), the order of the sentences to the seed."""
    b, ln = case["batch"], case["len"] if "len" in case else case["k_len"]
    order = torch.randperm(b, generator=gen, device="cuda")
    return torch.tensor(_mix(b, ln), dtype=torch.int32, device="cuda")[order].contiguous()


def _mix(b, ln):
    """b lengths at the even quantiles of a log-normal with median ln / 2, sigma 0.5; the longest is ln."""
    q = torch.special.ndtri((torch.arange(b, dtype=torch.float64) + 0.5) / b)
    v = torch.clamp(torch.round(0.5 * ln * torch.exp(0.5 * q)), 1, ln).to(torch.int64)
    v[-1] = ln
    return v.tolist()


def _randn(gen, shape, dt, std=1.0, mean=0.0):
    t = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    if std != 1.0:
        t.mul_(std)
    if mean:
        t.add_(mean)
    return t.to(DT[dt])


def _words(gen, shape, vocab):
    """Token ids distributed as words are: the rank-r word about as often as 1 / r."""
    u = torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)
    return torch.clamp(torch.exp(u * math.log(vocab)) - 1, 0, vocab - 1).to(torch.int32)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dt, kind = case["dt"], case["kind"]
    r = lambda shape, std=1.0, mean=0.0: _randn(gen, shape, dt, std, mean)  # noqa: E731
    t = {}
    if kind == "layer":
        B, Ln, N, D, F = case["batch"], case["len"], case["heads"], case["head_dim"], case["ffn"]
        H, T = N * D, B * Ln
        t["len"] = _lengths(case, gen)
        R = sum(_mix(B, Ln)) if case["packed"] else T
        t.update(qkv=r((T, 3 * H)), qkv_bias=r((3 * H,), 0.1), scores=r((B, N, Ln, Ln), math.sqrt(D)), ctx=r((B, N, Ln, D)),
                 res=r((R, H)), attn=r((R, H)), attn_bias=r((H,), 0.1), g1=r((H,), 0.1, 1.0), b1=r((H,), 0.1),
                 fc1=r((R, F)), fc1_bias=r((F,), 0.1), fc2=r((R, H)), fc2_bias=r((H,), 0.1), g2=r((H,), 0.1, 1.0), b2=r((H,), 0.1),
                 dy2=r((T, H)) if case["packed"] else r((R, H)), dres=r((R, H)), dact=r((R, F)), dy1=r((R, H)), dmerge=r((R, H)),
                 dprobs=r((B, N, Ln, Ln)), dq=r((B, N, Ln, D)), dk=r((B, N, Ln, D)), dv=r((B, N, Ln, D)))
    elif kind == "sublayer":
        T, H = case["rows"], case["hidden"]
        t.update(x=r((T, H)), bias=r((H,), 0.1), res=r((T, H)), gamma=r((H,), 0.1, 1.0), beta=r((H,), 0.1), dy=r((T, H)), dres=r((T, H)))
    elif kind == "softmax":
        shape = (case["batch"], case["heads"], case["q_len"], case["k_len"])
        t.update(x=r(shape, 8.0), dy=r(shape))
        t["len"] = _lengths(case, gen) if case["ragged"] else None
        # self-attention: padded queries are padding of the same sentences; cross-attention: the queries are another batch side
        t["qlen"] = t["len"] if case["ragged"] and case["q_len"] == case["k_len"] else None
    elif kind == "ffn":
        T, F = case["rows"], case["hidden"]
        t.update(x=r((T, F)), bias=r((F,), 0.1), dy=r((T, F)))
    elif kind == "heads":
        B, Ln, N, D, P = case["batch"], case["len"], case["heads"], case["head_dim"], case["parts"]
        t.update(x=r((B * Ln, P * N * D)), bias=r((P * N * D,), 0.1), ctx=r((B, N, Ln, D)), dctx=r((B * Ln, N * D)))
        t["d"] = [r((B, N, Ln, D)) for _ in range(P)]
    elif kind == "embedding":
        B, Ln, H, V = case["batch"], case["len"], case["hidden"], case["vocab"]
        tok = _words(gen, (B, Ln), V)
        if case["ragged"]:
            beyond = torch.arange(Ln, device="cuda")[None, :] >= _lengths(case, gen)[:, None]
            tok = torch.where(beyond, torch.full_like(tok, PAD), tok)
        t.update(tok=tok.contiguous(), emb=r((V, H), H ** -0.5), pos=r((Ln, H), 0.02), dy=r((B * Ln, H), 1e-2),
                 demb=r((V, H), 1e-2), dpos=r((Ln, H), 1e-2))      # gradients of an earlier micro-batch
    elif kind == "criterion":
        T, V = case["tokens"], case["vocab"]
        t["logits"] = torch.empty((T, V), dtype=DT[dt], device="cuda")
        for s in range(0, T, 1024):
            e = min(T, s + 1024)
            t["logits"][s:e] = r((e - s, V), 3.0)
        target = _words(gen, (T,), V)
        on = torch.randperm(T, generator=gen, device="cuda") < max(1, int(case["active"] * T))
        t["target"] = torch.where(on, target, torch.full_like(target, IGNORE))
    elif kind == "trainer":
        n = case["n"]
        t.update(p=_randn(gen, (n,), "f32", 0.02), m=_randn(gen, (n,), "f32", 1e-4), g=r((n,), 1e-3))
        t["v"] = torch.rand((n,), generator=gen, device="cuda", dtype=torch.float32).mul_(1e-6)
    elif kind == "padding":
        B, Ln, H = case["batch"], case["len"], case["hidden"]
        t.update(len=_lengths(case, gen), x=r((B, Ln, H)), packed=r((sum(_mix(B, Ln)), H)))
    return t


def prepare(case, seed):
    t = _inputs(case, seed)
    s = dict(case=case, t=t)
    if case["kind"] == "trainer":
        n, rule = case["n"], case["rule"]
        if rule in ("adam", "sgd"):
            t["p_lp"] = torch.empty(n, dtype=DT[case["dt"]], device="cuda")
        elif rule == "adam_blocked":
            t["state"] = L.lsq_adam_state_pack(t.pop("p"), t.pop("m"), t.pop("v"))
            t["p_lp"] = torch.empty(n, dtype=DT[case["dt"]], device="cuda")
        elif rule == "sgd_blocked":
            t["state"] = L.lsq_trainer_state_pack([t.pop("p"), t.pop("m")])
            t["p_lp"] = torch.empty(n, dtype=DT[case["dt"]], device="cuda")
        elif rule == "adam_lp":
            t["p_lp"] = t.pop("p").to(DT[case["dt"]])
        s["step"] = FIRST_STEP
    if case["graph"]:
        if case["kind"] == "embedding":      # the warm-up call below accumulates too: into copies
            kept = {k: t[k].clone() for k in ("demb", "dpos")}
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _CALLS[case["kind"]](case, t, s)
        torch.cuda.current_stream().wait_stream(side)
        if case["kind"] == "embedding":
            for k, v in kept.items():
                t[k].copy_(v)
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            s["out"] = _CALLS[case["kind"]](case, t, s)
    return s


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["out"]
    return _CALLS[state["case"]["kind"]](state["case"], state["t"], state)


# ------------------------------------------------------------------------------------------------- the calls
def _layer(case, t, s):
    B, Ln, N, D, p, act = case["batch"], case["len"], case["heads"], case["head_dim"], case["p"], case["act"]
    H, pa, scale, seed = N * D, case["p_attn"], case["head_dim"] ** -0.5, PHILOX_SEED
    packed = case["packed"]
    ql = t["len"] if packed else None
    o = {}
    o["q"], o["k"], o["v"] = L.lsq_split_heads_fwd(t["qkv"], t["qkv_bias"], B, Ln, N, D, 3)
    o["probs"], o["probs_drop"] = L.lsq_softmax_varlen_fwd(t["scores"], t["len"], ql, False, scale, pa, seed, 0)
    o["merged"] = L.lsq_merge_heads_fwd(t["ctx"])
    dy2 = t["dy2"]
    if packed:
        off = L.lsq_pad_offsets(t["len"], B, Ln)
        rows = t["res"].shape[0]
        o["offsets"], o["merged_packed"] = off, L.lsq_pad_remove(o["merged"].view(B, Ln, H), off, rows)
    o["h1"], o["y1"], o["mean1"], o["rstd1"] = L.lsq_bdr_layernorm_fwd(t["attn"], t["attn_bias"], t["res"], t["g1"], t["b1"], p, seed, 1, EPS)
    o["act"] = L.lsq_bias_act_dropout_fwd(t["fc1"], t["fc1_bias"], act, p, seed, 2)
    o["h2"], o["y2"], o["mean2"], o["rstd2"] = L.lsq_bdr_layernorm_fwd(t["fc2"], t["fc2_bias"], o["h1"], t["g2"], t["b2"], p, seed, 3, EPS)
    if packed:
        o["y2_padded"] = L.lsq_pad_restore(o["y2"], off, B, Ln)
        dy2 = o["dy2"] = L.lsq_pad_remove(t["dy2"].view(B, Ln, H), off, rows)
    o["dh2"], o["dx2"], o["dg2"], o["db2"], o["dbias2"] = L.lsq_bdr_layernorm_bwd(
        dy2, o["h2"], t["g2"], o["mean2"], o["rstd2"], p, seed, 3, t["dres"])
    o["dfc1"], o["dfc1_bias"] = L.lsq_bias_act_dropout_bwd(t["dact"], t["fc1"], t["fc1_bias"], act, p, seed, 2)
    o["dh1"], o["dx1"], o["dg1"], o["db1"], o["dbias1"] = L.lsq_bdr_layernorm_bwd(
        t["dy1"], o["h1"], t["g1"], o["mean1"], o["rstd1"], p, seed, 1, o["dh2"])
    dm = t["dmerge"]
    if packed:
        dm = o["dmerge"] = L.lsq_pad_restore(dm, off, B, Ln).view(B * Ln, H)
    o["dctx"] = L.lsq_merge_heads_bwd(dm, B, Ln, N, D)
    o["dscores"] = L.lsq_softmax_varlen_bwd(t["dprobs"], o["probs"], t["len"], ql, False, scale, pa, seed, 0)
    o["dqkv"], o["dqkv_bias"] = L.lsq_split_heads_bwd([t["dq"], t["dk"], t["dv"]], B, Ln, N, D)
    return o


def _sublayer(case, t, s):
    p, seed = case["p"], PHILOX_SEED
    o = {}
    if case["fused"]:
        o["h"], o["y"], o["mean"], o["rstd"] = L.lsq_bdr_layernorm_fwd(t["x"], t["bias"], t["res"], t["gamma"], t["beta"], p, seed, 1, EPS)
        o["dh"], o["dx"], o["dgamma"], o["dbeta"], o["dbias"] = L.lsq_bdr_layernorm_bwd(
            t["dy"], o["h"], t["gamma"], o["mean"], o["rstd"], p, seed, 1, t["dres"])
    else:
        o["h"] = L.lsq_bias_dropout_residual_fwd(t["x"], t["bias"], t["res"], p, seed, 1)
        o["y"], o["mean"], o["rstd"] = L.lsq_layernorm_fwd(o["h"], t["gamma"], t["beta"], EPS)
        o["dh"], o["dgamma"], o["dbeta"] = L.lsq_layernorm_bwd(t["dy"], o["h"], t["gamma"], o["mean"], o["rstd"], t["dres"])
        o["dx"], o["dbias"] = L.lsq_bias_dropout_residual_bwd(o["dh"], p, seed, 1)
    return o


def _softmax(case, t, s):
    a = (case["causal"], 0.125, case["p_attn"], PHILOX_SEED, 0)
    if t["qlen"] is not None:
        y, yd = L.lsq_softmax_varlen_fwd(t["x"], t["len"], t["qlen"], *a)
        dx = L.lsq_softmax_varlen_bwd(t["dy"], y, t["len"], t["qlen"], *a)
    else:
        y, yd = L.lsq_softmax_fwd(t["x"], t["len"], *a)
        dx = L.lsq_softmax_bwd(t["dy"], y, t["len"], *a)
    return dict(y=y, y_drop=yd, dx=dx)


def _ffn(case, t, s):
    a = (case["act"], case["p"], PHILOX_SEED, 2)
    out = L.lsq_bias_act_dropout_fwd(t["x"], t["bias"], *a)
    dx, dbias = L.lsq_bias_act_dropout_bwd(t["dy"], t["x"], t["bias"], *a)
    return dict(out=out, dx=dx, dbias=dbias)


def _heads(case, t, s):
    B, Ln, N, D, P = case["batch"], case["len"], case["heads"], case["head_dim"], case["parts"]
    parts = L.lsq_split_heads_fwd(t["x"], t["bias"], B, Ln, N, D, P)
    merged = L.lsq_merge_heads_fwd(t["ctx"])
    dctx = L.lsq_merge_heads_bwd(t["dctx"], B, Ln, N, D)
    dx, dbias = L.lsq_split_heads_bwd(t["d"], B, Ln, N, D)
    return dict(parts=list(parts), merged=merged, dctx=dctx, dx=dx, dbias=dbias)


def _embedding(case, t, s):
    a = (PAD, math.sqrt(case["hidden"]), case["p"], PHILOX_SEED, 5)
    out = L.lsq_embedding_fwd(t["tok"], t["emb"], t["pos"], *a)
    L.lsq_embedding_bwd(t["demb"], t["dpos"], t["dy"], t["tok"], *a)
    return dict(out=out, demb=t["demb"], dpos=t["dpos"])


def _criterion(case, t, s):
    a = (case["alpha"], IGNORE)
    if case["one_pass"]:
        loss, nll, lse, sums, dl = L.lsq_ls_xent_fwd_bwd(t["logits"], t["target"], *a, 1.0)
    else:
        loss, nll, lse, sums = L.lsq_ls_xent_fwd(t["logits"], t["target"], *a)
        dl = L.lsq_ls_xent_bwd(t["logits"], lse, t["target"], *a, 1.0)
    return dict(loss=loss, nll=nll, lse=lse, sums=sums, dlogits=dl)


def _trainer(case, t, s):
    rule = case["rule"]
    s["step"] += 1
    if rule == "adam":
        return L.lsq_adam_step(t["p"], t["m"], t["v"], t["g"], t["p_lp"], step=s["step"], **ADAM)
    if rule == "adam_blocked":
        return L.lsq_adam_step_blocked(t["state"], t["g"], t["p_lp"], step=s["step"], **ADAM)
    if rule == "adam_lp":
        return L.lsq_adam_step_lp(t["p_lp"], t["m"], t["v"], t["g"], step=s["step"], **ADAM)
    if rule == "sgd":
        return L.lsq_sgd_step(t["p"], t["m"], t["g"], t["p_lp"], **SGD)
    return L.lsq_sgd_step_blocked(t["state"], t["g"], t["p_lp"], **SGD)


def _padding(case, t, s):
    B, Ln = case["batch"], case["len"]
    off = L.lsq_pad_offsets(t["len"], B, Ln)
    packed = L.lsq_pad_remove(t["x"], off, t["packed"].shape[0])
    padded = L.lsq_pad_restore(t["packed"], off, B, Ln)
    return dict(offsets=off, packed=packed, padded=padded)


_CALLS = dict(layer=_layer, sublayer=_sublayer, softmax=_softmax, ffn=_ffn, heads=_heads, embedding=_embedding,
              criterion=_criterion, trainer=_trainer, padding=_padding)


# -------------------------------------------------------------------------------------------------------- work
def work(case):
    """Bytes and operations of one pass: every call's inputs read once and its outputs written once (a tensor that the
    forward saves is read again by the backward, which runs much later in a program); masked scores are not read."""
    e, kind = SIZE[case["dt"]], case["kind"]
    if kind == "layer":
        B, Ln, F = case["batch"], case["len"], case["ffn"]
        H, T = case["heads"] * case["head_dim"], B * Ln
        mix = _mix(B, Ln)
        R = sum(mix) if case["packed"] else T
        sm = _softmax_work(B, case["heads"], Ln, Ln, False, mix, mix if case["packed"] else None, case["p_attn"] > 0, e)
        moved = 2 * 3 * T * H * 2 + 2 * T * H * 2 + 2 * (4 + 5) * R * H + 5 * R * F
        if case["packed"]:
            moved += 2 * (2 * R * H) + 2 * (R + T) * H
        return dict(bytes=e * moved + sm["bytes"], flops=40.0 * R * H + 20.0 * R * F + sm["flops"])
    if kind == "sublayer":
        n = case["rows"] * case["hidden"]
        return dict(bytes=e * n * (9 if case["fused"] else 11) + 16 * case["rows"], flops=35.0 * n)
    if kind == "softmax":
        mix = _mix(case["batch"], case["k_len"]) if case["ragged"] else None
        return _softmax_work(case["batch"], case["heads"], case["q_len"], case["k_len"], case["causal"], mix,
                             mix if case["q_len"] == case["k_len"] else None, case["p_attn"] > 0, e)
    if kind == "ffn":
        n = case["rows"] * case["hidden"]
        return dict(bytes=5 * e * n, flops=(40.0 if case["act"] != "relu" else 8.0) * n)
    if kind == "heads":
        n = case["batch"] * case["len"] * case["heads"] * case["head_dim"]
        return dict(bytes=4 * e * n * (case["parts"] + 1), flops=2.0 * n * case["parts"])
    if kind == "embedding":
        n = case["batch"] * case["len"] * case["hidden"]
        if case["ragged"]:
            n = int(n * sum(_mix(case["batch"], case["len"])) / (case["batch"] * case["len"]))
        # table rows read, out written; dy read, each touched gradient row read and written once (about half the tokens are repeats)
        return dict(bytes=e * n * 3 + e * n, flops=6.0 * n)
    if kind == "criterion":
        T, V = case["tokens"], case["vocab"]
        active = max(1, int(case["active"] * T))
        return dict(bytes=e * V * (active * (1 if case["one_pass"] else 2) + T) + 20 * T, flops=8.0 * active * V)
    if kind == "trainer":
        n, rule = case["n"], case["rule"]
        each = {"adam": 28, "adam_blocked": 28, "adam_lp": 22, "sgd": 20, "sgd_blocked": 20}[rule]
        return dict(bytes=each * n, flops=15.0 * n)
    B, Ln, H = case["batch"], case["len"], case["hidden"]
    R = sum(_mix(B, Ln))
    return dict(bytes=e * H * (3 * R + B * Ln), flops=0.0)


def _softmax_work(B, N, Lq, Lk, causal, klen, qlen, drop, e):
    allowed = 0
    for b in range(B):
        kl = Lk if klen is None else klen[b]
        i = torch.arange(Lq if qlen is None else qlen[b])
        allowed += int(torch.clamp(i + 1 + Lk - Lq, 0, kl).sum()) if causal else kl * len(i)
    total = B * N * Lq * Lk
    return dict(bytes=e * (3 * N * allowed + total * (3 if drop else 2)), flops=15.0 * N * allowed)


def tolerance(case):
    """Relative error of an output whose sums run in another order or whose roundings fall elsewhere, four times what
    the outputs differ by from 64-bit results on this machine: the storage type's rounding (f16 2e-4..3e-4, bf16 1.6e-3..2.4e-3 of a
    result's norm), or that of 32-bit sums."""
    if case["kind"] == "padding":
        return "exact"
    if case["kind"] == "trainer":            # 32-bit state; a rounding that falls elsewhere moves a 16-bit copy by one place, seldom
        return {"rel": {"f16": 2e-5, "bf16": 1e-4}[case["dt"]], "max": {"f16": 2e-3, "bf16": 1.6e-2}[case["dt"]]}
    return {"rel": {"f32": 1e-5, "f16": 1.2e-3, "bf16": 1e-2}[case["dt"]]}


# ------------------------------------------------------------------------------------------ 64-bit references
def _philox(n, offset):
    """16-bit lane of every element e < n: Philox4x32-10 of counter (e / 8, offset), lane e % 8."""
    g = torch.arange((n + 7) // 8, dtype=torch.int64, device="cuda")
    lo = 0xFFFFFFFF
    c = [g & lo, g >> 32, torch.full_like(g, offset & lo), torch.full_like(g, offset >> 32)]
    k0, k1 = PHILOX_SEED & lo, PHILOX_SEED >> 32
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57          # wraps mod 2^64: the bits are right
        c = [((b >> 32) & lo) ^ c[1] ^ k0, b & lo, ((a >> 32) & lo) ^ c[3] ^ k1, a & lo]
        k0, k1 = (k0 + 0x9E3779B9) & lo, (k1 + 0xBB67AE85) & lo
    return torch.stack([(w >> s) & 0xFFFF for w in c for s in (0, 16)], dim=1).reshape(-1)[:n]


def _keep(shape, p, offset):
    """keep / (1 - p) as float64, or 1."""
    if p == 0:
        return 1.0
    n = math.prod(shape)
    return (_philox(n, offset) >= int(round(p * 65536))).reshape(shape).double() / (1.0 - p)


def _x_ln(h, g, b):
    mean = h.mean(1)
    rstd = torch.rsqrt(h.var(1, unbiased=False) + EPS)
    return (h - mean[:, None]) * rstd[:, None] * g + b, mean, rstd


def _x_ln_bwd(dy, h, g, mean, rstd, dres):
    xh = (h - mean[:, None]) * rstd[:, None]
    gy = g * dy
    dh = rstd[:, None] * (gy - gy.mean(1, keepdim=True) - xh * (gy * xh).mean(1, keepdim=True)) + dres
    return dh, (dy * xh).sum(0), dy.sum(0)


def _x_act(z, act):
    """act(z), act'(z)"""
    if act == "relu":
        return torch.clamp(z, min=0), (z > 0).double()
    if act == "gelu":
        c = torch.special.ndtr(z)
        return z * c, c + z * torch.exp(-0.5 * z * z) / math.sqrt(2 * math.pi)
    k = math.sqrt(2 / math.pi)
    th = torch.tanh(k * (z + 0.044715 * z ** 3))
    return 0.5 * z * (1 + th), 0.5 * (1 + th) + 0.5 * z * (1 - th * th) * k * (1 + 3 * 0.044715 * z * z)


def _x_softmax(x, dy, klen, qlen, causal, scale, p):
    B, N, Lq, Lk = x.shape
    on = torch.ones((B, 1, Lq, Lk), dtype=torch.bool, device="cuda")
    j = torch.arange(Lk, device="cuda")
    i = torch.arange(Lq, device="cuda")
    if klen is not None:
        on &= j[None, None, None, :] < klen[:, None, None, None]
    if qlen is not None:
        on &= i[None, None, :, None] < qlen[:, None, None, None]
    if causal:
        on &= j[None, :] <= i[:, None] + (Lk - Lq)
    y = torch.softmax(torch.where(on, x.double() * scale, torch.full((), -math.inf, dtype=torch.float64, device="cuda")), -1)
    y = torch.where(on, y, torch.zeros((), dtype=torch.float64, device="cuda"))
    keep = _keep(x.shape, p, 0)
    yd = y * keep if p > 0 else None
    dy = dy.double() * keep
    dx = scale * y * (dy - (torch.where(on, dy, 0.0) * y).sum(-1, keepdim=True))
    return y, yd, torch.where(on, dx, 0.0)


def _split(x, B, Ln, N, D, P):
    return [v.contiguous() for v in x.reshape(B, Ln, P, N, D).permute(2, 0, 3, 1, 4)]


def _join(parts, B, Ln):
    return torch.stack(parts, 0).permute(1, 3, 0, 2, 4).reshape(B * Ln, -1)


def exact(case, seed):
    kind, p = case["kind"], case.get("p", 0.0)
    t = _inputs(case, seed)
    d = {k: v.double() for k, v in t.items() if torch.is_tensor(v) and v.is_floating_point() and kind not in ("softmax", "criterion", "trainer")}
    if kind == "layer":
        B, Ln, N, D = case["batch"], case["len"], case["heads"], case["head_dim"]
        H, packed = N * D, case["packed"]
        real = (torch.arange(Ln, device="cuda")[None, :] < t["len"][:, None]).reshape(-1)
        o = dict(zip("qkv", _split(d["qkv"] + d["qkv_bias"], B, Ln, N, D, 3)))
        o["probs"], o["probs_drop"], o["dscores"] = _x_softmax(t["scores"], t["dprobs"], t["len"], t["len"] if packed else None, False,
                                                               D ** -0.5, case["p_attn"])
        o["merged"] = _join([d["ctx"]], B, Ln)
        o["h1"] = d["res"] + _keep(d["res"].shape, p, 1) * (d["attn"] + d["attn_bias"])
        o["y1"], o["mean1"], o["rstd1"] = _x_ln(o["h1"], d["g1"], d["b1"])
        a, slope = _x_act(d["fc1"] + d["fc1_bias"], case["act"])
        keep = _keep(a.shape, p, 2)
        o["act"], o["dfc1"] = keep * a, keep * slope * d["dact"]
        o["dfc1_bias"] = o["dfc1"].sum(0)
        keep2 = _keep(d["res"].shape, p, 3)
        o["h2"] = o["h1"] + keep2 * (d["fc2"] + d["fc2_bias"])
        o["y2"], o["mean2"], o["rstd2"] = _x_ln(o["h2"], d["g2"], d["b2"])
        dy2, dm = d["dy2"], d["dmerge"]
        if packed:
            o["offsets"] = None
            o["merged_packed"] = o["merged"][real]
            o["y2_padded"] = torch.zeros((B * Ln, H), dtype=torch.float64, device="cuda")
            o["y2_padded"][real] = o["y2"]
            o["y2_padded"] = o["y2_padded"].view(B, Ln, H)
            dy2 = o["dy2"] = dy2[real]
            o["dmerge"] = torch.zeros((B * Ln, H), dtype=torch.float64, device="cuda")
            o["dmerge"][real] = dm
            dm = o["dmerge"]
        o["dh2"], o["dg2"], o["db2"] = _x_ln_bwd(dy2, o["h2"], d["g2"], o["mean2"], o["rstd2"], d["dres"])
        o["dx2"] = keep2 * o["dh2"]
        o["dh1"], o["dg1"], o["db1"] = _x_ln_bwd(d["dy1"], o["h1"], d["g1"], o["mean1"], o["rstd1"], o["dh2"])
        o["dx1"] = _keep(d["res"].shape, p, 1) * o["dh1"]
        o["dbias2"], o["dbias1"] = o["dx2"].sum(0), o["dx1"].sum(0)
        o["dctx"] = _split(dm, B, Ln, N, D, 1)[0]
        o["dqkv"] = _join([d["dq"], d["dk"], d["dv"]], B, Ln)
        o["dqkv_bias"] = o["dqkv"].sum(0)
        return o
    if kind == "sublayer":
        keep = _keep(d["x"].shape, p, 1)
        h = d["res"] + keep * (d["x"] + d["bias"])
        y, mean, rstd = _x_ln(h, d["gamma"], d["beta"])
        dh, dg, db = _x_ln_bwd(d["dy"], h, d["gamma"], mean, rstd, d["dres"])
        dx = keep * dh
        return dict(h=h, y=y, mean=mean, rstd=rstd, dh=dh, dx=dx, dgamma=dg, dbeta=db, dbias=dx.sum(0))
    if kind == "softmax":
        y, yd, dx = _x_softmax(t["x"], t["dy"], t["len"], t["qlen"], case["causal"], 0.125, case["p_attn"])
        return dict(y=y, y_drop=yd, dx=dx)
    if kind == "ffn":
        a, slope = _x_act(d["x"] + d["bias"], case["act"])
        keep = _keep(a.shape, p, 2)
        dx = keep * slope * d["dy"]
        return dict(out=keep * a, dx=dx, dbias=dx.sum(0))
    if kind == "heads":
        B, Ln, N, D, P = case["batch"], case["len"], case["heads"], case["head_dim"], case["parts"]
        dx = _join([v.double() for v in t["d"]], B, Ln)
        return dict(parts=_split(d["x"] + d["bias"], B, Ln, N, D, P), merged=_join([d["ctx"]], B, Ln),
                    dctx=_split(d["dctx"], B, Ln, N, D, 1)[0], dx=dx, dbias=dx.sum(0))
    if kind == "embedding":
        B, Ln, H = case["batch"], case["len"], case["hidden"]
        tok = t["tok"].reshape(-1).long()
        real = (tok != PAD).double()[:, None]
        keep = _keep((B * Ln, H), p, 5) * real
        out = keep * (math.sqrt(H) * d["emb"][tok] + d["pos"].repeat(B, 1))
        dk = keep * d["dy"]
        demb = d["demb"].index_add(0, tok, dk * math.sqrt(H))
        return dict(out=out, demb=demb, dpos=d["dpos"] + dk.view(B, Ln, H).sum(0))
    if kind == "criterion":
        T, V, alpha = case["tokens"], case["vocab"], case["alpha"]
        on, k = t["target"] != IGNORE, torch.clamp(t["target"], min=0).long()
        o = dict(loss=torch.zeros(T, dtype=torch.float64, device="cuda"))
        o["nll"], o["lse"] = torch.zeros_like(o["loss"]), torch.zeros_like(o["loss"])
        o["dlogits"] = torch.zeros((T, V), dtype=torch.float64, device="cuda")
        for s in range(0, T, 512):
            e = min(T, s + 512)
            h, w, kk = t["logits"][s:e].double(), on[s:e].double(), k[s:e, None]
            lse = torch.logsumexp(h, 1)
            hk = h.gather(1, kk)[:, 0]
            o["lse"][s:e], o["nll"][s:e] = lse * w, (lse - hk) * w
            o["loss"][s:e] = (lse - (1 - alpha) * hk - alpha / V * h.sum(1)) * w
            dl = torch.exp(h - lse[:, None]) - alpha / V
            dl.scatter_add_(1, kk, torch.full_like(kk, -(1 - alpha), dtype=torch.float64))
            o["dlogits"][s:e] = dl * w[:, None]
        o["sums"] = torch.stack([o["loss"].sum(), o["nll"].sum(), on.sum().double()])
        return o
    if kind == "trainer":
        rule, step = case["rule"], FIRST_STEP + 1
        p0 = (t["p"].to(DT[case["dt"]]) if rule == "adam_lp" else t["p"]).double()
        m, v, g = t["m"].double(), t["v"].double(), t["g"].double()
        if rule in ("sgd", "sgd_blocked"):
            m = SGD["momentum"] * m + g
            q = p0 - SGD["lr"] * m
            return (q, m, q) if rule == "sgd" else None
        b1, b2 = ADAM["beta1"], ADAM["beta2"]
        m, v = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
        q = p0 - ADAM["lr"] * (m / (1 - b1 ** step)) / (torch.sqrt(v / (1 - b2 ** step)) + ADAM["eps"])
        return {"adam": (q, m, v, q), "adam_lp": (q, m, v), "adam_blocked": (None, q)}[rule]
    return None
