"""The work that users of this framework have it do, as cases to be timed and compared.

Every case is one pass through the public entry points, with inputs made on
the GPU from a seed:

* ``model``       runtime.Model.train_step: embedding, layers, loss head,
                  backward, gradient-norm clip and AdamW of a whole model;
* ``layer``       one decoder layer (dense or routed experts): forward and
                  backward over one or more micro-batches, or, with ``adamw``,
                  forward and the backward with its fused optimizer updates;
* ``attention``   causal grouped-query attention forward and backward;
* ``head``        final norm, LM head and cross-entropy, forward and backward;
* ``projection``  the three products of one projection (y, dx, dw);
* ``routing``     top-k routing and the expert-major permutation.

``exact`` recomputes a case in float64 with plain torch.
"""
import math

import numpy as np
import torch

from paper_2609_13645_amd import _lib, runtime

DEV = "cuda"
BETA1, BETA2, ADAM_EPS, WEIGHT_DECAY, LR = 0.9, 0.95, 1e-8, 0.1, 1e-5
STEP = 100  # optimizer steps behind a case's optimizer state

_LAYER = dict(batch=1, seq=128, hidden=256, n_heads=4, n_kv_heads=2, head_dim=64, ffn=0,
              rope_base=10000.0, rms_eps=1e-5, n_experts=0, top_k=0, expert_ffn=0, shared_ffn=0,
              aux_coef=0.0, recompute_attn=0, qk_norm=0, branch_scale=0.0)


def _layer(name, **kw):
    extra = dict(kind="layer", micro=1, adamw=False, packed=False)
    c = dict(_LAYER, **extra)
    c.update(kw)
    return dict(c, name=name) if name else c


def _model(name, **kw):
    c = dict(_LAYER, kind="model", vocab=1024, n_layers=1, tied=False)
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest training step: one short sequence through a one-layer
        # model; launches and latency are all of it
        _model("tiny_model_step", ffn=688),
        # a whole model's step at ordinary widths (head dim 64, tied head),
        # two layers of it
        _model("dense_model_step", batch=2, seq=1024, hidden=2048, n_heads=32, n_kv_heads=8,
               ffn=8192, vocab=32000, n_layers=2, tied=True),
        # a small layer on ragged sequences, gradients accumulated over two
        # micro-batches
        _layer("small_layer_accumulated", batch=3, seq=333, hidden=768, n_heads=12, n_kv_heads=4,
               ffn=2056, micro=2),
        # QK-Norm layer of a small model at a long batch: many tokens, narrow
        # products
        _layer("qk_norm_layer", batch=4, seq=4096, hidden=1024, n_heads=16, n_kv_heads=8,
               head_dim=128, ffn=3072, rope_base=1e6, rms_eps=1e-6, qk_norm=1),
        # the headline training step: 8B-shape layer, forward, backward and
        # optimizer
        _layer("llama8b_layer_step", seq=4096, hidden=4096, n_heads=32, n_kv_heads=8,
               head_dim=128, ffn=14336, rope_base=500000.0, adamw=True),
        # the largest call: the same layer on a 16K sequence, attention
        # recomputed in the backward
        _layer("llama8b_layer_16k", seq=16384, hidden=4096, n_heads=32, n_kv_heads=8,
               head_dim=128, ffn=14336, rope_base=500000.0, recompute_attn=1),
        # routed experts at full size, with the optimizer step of their
        # weights
        _layer("moe_layer_step", batch=2, seq=4096, hidden=2048, n_heads=16, n_kv_heads=4,
               head_dim=128, n_experts=64, top_k=8, expert_ffn=1408, aux_coef=1e-2, adamw=True),
        # many small experts on a short odd sequence: about a hundred rows
        # per expert, two kv heads, a shared expert
        _layer("many_expert_layer_short", seq=1000, hidden=2048, n_heads=32, n_kv_heads=2,
               head_dim=128, n_experts=160, top_k=16, expert_ffn=512, shared_ffn=512,
               aux_coef=1e-2, rms_eps=1e-6, branch_scale=1.4 / 28 ** 0.5),
        # attention alone at head dim 64, sequences that end inside a tile
        dict(name="attention_d64", kind="attention", batch=4, seq=2047, n_heads=32, n_kv_heads=8,
             head_dim=64),
        # the loss head of a 32k-vocabulary model on an odd number of tokens
        dict(name="loss_head", kind="head", tokens=4095, hidden=2048, vocab=32000, chunk=0,
             logit_scale=0.0),
        # a projection's three products at a size between the tile shapes
        dict(name="projection", kind="projection", tokens=1000, n_out=3072, n_in=1024),
        # token routing as a call of its own
        dict(name="routing", kind="routing", tokens=8192, n_experts=64, top_k=8),
    ]


# ------------------------------------------------------------------ draw ----

def _log(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    return max(lo, min(hi, int(v) // step * step))


def _heads(rng, hidden):
    """Heads whose total width is between half and twice the hidden width."""
    while True:
        kv, group, d = rng.choice((1, 2, 4, 8)), rng.choice((1, 2, 4, 8)), rng.choice((64, 128))
        if kv * group <= 32 and hidden <= 2 * kv * group * d <= 4 * hidden:
            return dict(n_heads=kv * group, n_kv_heads=kv, head_dim=d)


def draw(rng):
    kind = rng.choice(("model", "layer", "layer", "moe", "attention", "head", "projection",
                       "routing"))
    if kind == "model":
        h = _log(rng, 256, 2048, 64)
        return _model(None, batch=rng.randint(1, 4), seq=_log(rng, 64, 1024), hidden=h,
                      **_heads(rng, h), ffn=_log(rng, 2 * h, 4 * h, 8),
                      vocab=_log(rng, 1000, 32000, 8), n_layers=rng.randint(1, 2),
                      tied=rng.random() < 0.5)
    if kind == "layer":
        h = _log(rng, 256, 4096, 8)
        adamw = rng.random() < 0.4
        return _layer(None, batch=rng.randint(1, 4), seq=_log(rng, 64, 4096), hidden=h,
                      **_heads(rng, h), ffn=_log(rng, 2 * h, 4 * h, 8),
                      qk_norm=int(rng.random() < 0.3), recompute_attn=int(rng.random() < 0.2),
                      packed=rng.random() < 0.3, adamw=adamw,
                      micro=1 if adamw else rng.randint(1, 2))
    if kind == "moe":
        E, k = rng.choice(((8, 2), (16, 4), (64, 8), (160, 16)))
        h = _log(rng, 512, 2048, 64)
        return _layer(None, batch=rng.randint(1, 2), seq=_log(rng, 128, 4096), hidden=h,
                      **_heads(rng, h), n_experts=E, top_k=k,
                      expert_ffn=_log(rng, 128, 1408, 8),
                      shared_ffn=rng.choice((0, 0, 512)), aux_coef=1e-2,
                      adamw=rng.random() < 0.5)
    if kind == "attention":
        return dict(kind=kind, batch=rng.randint(1, 4), seq=_log(rng, 64, 4096),
                    **_heads(rng, _log(rng, 256, 4096)))
    if kind == "head":
        return dict(kind=kind, tokens=_log(rng, 64, 4096), hidden=_log(rng, 256, 4096, 8),
                    vocab=_log(rng, 1000, 32000, 8), chunk=rng.choice((0, 0, 1024)),
                    logit_scale=rng.choice((0.0, 0.25)))
    if kind == "projection":
        return dict(kind=kind, tokens=_log(rng, 64, 8192, 8), n_out=_log(rng, 128, 8192, 8),
                    n_in=_log(rng, 128, 8192, 8))
    E, k = rng.choice(((8, 2), (16, 4), (64, 8), (160, 16)))
    return dict(kind="routing", tokens=_log(rng, 64, 16384), n_experts=E, top_k=k)


# ---------------------------------------------------------------- inputs ----

class _Draw:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, shape, std, mean=0.0):
        return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(mean, std,
                                                                           generator=self.g)

    def bf16(self, shape, std, mean=0.0):
        return self.normal(shape, std, mean).to(torch.bfloat16)

    def uniform(self, shape, lo, hi):
        return torch.empty(shape, dtype=torch.float32, device=DEV).uniform_(lo, hi,
                                                                            generator=self.g)

    def ints(self, n, hi):
        return torch.randint(0, hi, (n,), generator=self.g, device=DEV, dtype=torch.int32)


def _layer_weights(d, c):
    return {n: d.bf16(s, 0.1, 1.0) if len(s) == 1 else d.bf16(s, 0.02)
            for n, s in runtime.layer_shapes(c).items()}


def _layer_x(d, c, w):
    """Input activations. Tokens of a routed layer lean towards the router
    rows of the experts they belong to, as a trained router's tokens do: its
    choice is clear of the rounding of the logits. The experts are not
    equally popular."""
    T = c["batch"] * c["seq"]
    x = d.normal((T, c["hidden"]), 1.0)
    if c["n_experts"]:
        rows = w["w_router"].float()
        rows = rows / rows.norm(dim=1, keepdim=True)
        taste = d.normal((c["n_experts"],), 0.3) - torch.log(
            -torch.log(d.uniform((T, c["n_experts"]), 1e-6, 1.0 - 1e-6)))
        chosen = taste.topk(c["top_k"], dim=1).indices
        x += 10.0 * torch.zeros_like(taste).scatter_(1, chosen, 1.0) @ rows
    return x.to(torch.bfloat16)


def _positions(d, c):
    """RoPE positions of rows packed with documents of 1 to 512 tokens."""
    T = c["batch"] * c["seq"]
    starts = d.uniform((T,), 0.0, 1.0) < 1.0 / 256.0
    i = torch.arange(T, device=DEV)
    starts |= i % c["seq"] == 0
    return (i - torch.where(starts, i, 0).cummax(0).values).to(torch.int32)


def _moments(d, n, scale):
    return d.normal((n,), scale), d.uniform((n,), 0.5, 1.5) * scale ** 2


def _layer_inputs(c, seed):
    d = _Draw(seed)
    T, w = c["batch"] * c["seq"], _layer_weights(d, c)
    i = dict(w=w, x=[], dy=[])
    for _ in range(c["micro"]):
        i["x"].append(_layer_x(d, c, w))
        i["dy"].append(d.bf16((T, c["hidden"]), 1e-2))
    i["positions"] = _positions(d, c) if c["packed"] else None
    i["moments"] = {n: _moments(d, t.numel(), 1e-2) for n, t in w.items()} if c["adamw"] else None
    return i


def _model_inputs(c, seed):
    d = _Draw(seed)
    V, h, T = c["vocab"], c["hidden"], c["batch"] * c["seq"]
    i = dict(embedding=d.bf16((V, h), 0.02), final_norm=d.bf16((h,), 0.1, 1.0),
             w_lm=None if c["tied"] else d.bf16((V, h), 0.02),
             layers=[_layer_weights(d, c) for _ in range(c["n_layers"])])
    i.update(ids=d.ints(T, V), targets=d.ints(T, V))
    tensors = [i["embedding"], i["final_norm"]] + ([] if c["tied"] else [i["w_lm"]])
    n = sum(t.numel() for t in tensors) + sum(t.numel() for w in i["layers"] for t in w.values())
    i["moment_draw"], i["moment_scale"] = d, n ** -0.5
    return i


def _model_names(c):
    names = ["embedding", "final_norm"] + ([] if c["tied"] else ["w_lm"])
    return names + [f"{l}.{n}" for l in range(c["n_layers"]) for n in runtime.layer_shapes(c)]


def _bits(t):
    return None if t is None else t.view(torch.int16).cpu().numpy().view(np.uint16)


# --------------------------------------------------------------- prepare ----

def prepare(case, seed):
    return {"model": _prepare_model, "layer": _prepare_layer, "attention": _prepare_attention,
            "head": _prepare_head, "projection": _prepare_projection,
            "routing": _prepare_routing}[case["kind"]](case, seed)


def _optimizer_scalars():
    scalars = torch.tensor([LR, 0.0, 0.0, 1.0], dtype=torch.float32, device=DEV)
    return scalars, torch.full((1,), STEP, dtype=torch.int32, device=DEV)


def _prepare_model(c, seed):
    i = _model_inputs(c, seed)
    cfg = dict(c, lr=LR, beta1=BETA1, beta2=BETA2, adam_eps=ADAM_EPS, weight_decay=WEIGHT_DECAY)
    m = runtime.Model(cfg, dict(
        embedding=_bits(i["embedding"]), final_norm=_bits(i["final_norm"]), w_lm=_bits(i["w_lm"]),
        layers=[{n: _bits(t) for n, t in w.items()} for w in i["layers"]],
        ids=i["ids"].cpu().numpy(), targets=i["targets"].cpu().numpy()))
    f = m.flat
    for n in _model_names(c):
        mom, var = _moments(i["moment_draw"], f.view(f.m, n).numel(), i["moment_scale"])
        f.view(f.m, n).copy_(mom.view(f.offsets[n][1]))
        f.view(f.v, n).copy_(var.view(f.offsets[n][1]))
    m.dev_step.fill_(STEP)
    return dict(kind="model", model=m, names=_model_names(c))


def _prepare_layer(c, seed):
    i = _layer_inputs(c, seed)
    cfg = dict(c)
    if i["positions"] is not None:
        cfg["positions"] = i["positions"].cpu().numpy()
    bits = {n: _bits(t) for n, t in i["w"].items()}
    s = dict(kind="layer", x=i["x"], dy=i["dy"], adamw=c["adamw"], moe=c["n_experts"] > 0)
    if c["adamw"]:
        f = s["flat"] = runtime.FlatParams(runtime.layer_shapes(c))
        s["layer"] = runtime.Layer(cfg, bits, flat=f)
        for n, (mom, var) in i["moments"].items():
            f.view(f.m, n).copy_(mom.view(f.offsets[n][1]))
            f.view(f.v, n).copy_(var.view(f.offsets[n][1]))
        s["scalars"], s["step"] = _optimizer_scalars()
        s["hp"] = _lib.AdamwHparams(BETA1, BETA2, ADAM_EPS, WEIGHT_DECAY)
    else:
        s["layer"] = runtime.Layer(cfg, bits)
    s["out"] = [torch.empty_like(x) for x in i["x"]]
    s["dx"] = [torch.empty_like(x) for x in i["x"]]
    return s


def _attention_inputs(c, seed):
    d = _Draw(seed)
    T, hq, hkv = c["batch"] * c["seq"], c["n_heads"] * c["head_dim"], c["n_kv_heads"] * c["head_dim"]
    return d.bf16((T, hq + 2 * hkv), 1.0), d.bf16((T, hq), 1.0)


def _prepare_attention(c, seed):
    qkv, do = _attention_inputs(c, seed)
    a = _lib.attn_cfg(c)
    return dict(kind="attention", cfg=a, qkv=qkv, do=do, o=torch.empty_like(do),
                lse=torch.empty((c["batch"], c["n_heads"], c["seq"]), dtype=torch.float32,
                                device=DEV),
                dqkv=torch.empty_like(qkv),
                ws=runtime.empty_bytes(_lib.forge_attention_bwd_workspace_bytes(a)))


def _head_inputs(c, seed):
    d = _Draw(seed)
    T, h, V = c["tokens"], c["hidden"], c["vocab"]
    return dict(x=d.bf16((T, h), 1.0), g=d.bf16((h,), 0.1, 1.0), w=d.bf16((V, h), 0.02),
                targets=d.ints(T, V))


def _prepare_head(c, seed):
    i = _head_inputs(c, seed)
    cfg = _lib.HeadCfg(c["tokens"], c["hidden"], c["vocab"], 1e-5, c["logit_scale"])
    ws = (_lib.forge_loss_chunked_workspace_bytes(cfg, c["chunk"]) if c["chunk"]
          else _lib.forge_loss_workspace_bytes(cfg))
    return dict(i, kind="head", cfg=cfg, chunk=c["chunk"], ws=runtime.empty_bytes(ws),
                loss=torch.zeros(1, dtype=torch.float32, device=DEV), dx=torch.empty_like(i["x"]),
                dg=torch.zeros(i["g"].shape, dtype=torch.float32, device=DEV),
                dw=torch.zeros(i["w"].shape, dtype=torch.float32, device=DEV))


def _projection_inputs(c, seed):
    d = _Draw(seed)
    T, n, k = c["tokens"], c["n_out"], c["n_in"]
    return d.bf16((T, k), 1.0), d.bf16((n, k), 0.02), d.bf16((T, n), 1e-2)


def _prepare_projection(c, seed):
    x, w, dy = _projection_inputs(c, seed)
    return dict(kind="projection", x=x, w=w, dy=dy, y=torch.empty_like(dy),
                dx=torch.empty_like(x), dw=torch.empty(w.shape, dtype=torch.float32, device=DEV))


def _prepare_routing(c, seed):
    T, E, k = c["tokens"], c["n_experts"], c["top_k"]

    def ints(*shape):
        return torch.empty(shape, dtype=torch.int32, device=DEV)

    return dict(kind="routing", T=T, E=E, k=k, logits=_Draw(seed).normal((T, E), 1.0),
                idx=ints(T, k), gates=torch.empty((T, k), dtype=torch.float32, device=DEV),
                probs=torch.empty((T, E), dtype=torch.float32, device=DEV), counts=ints(E),
                offsets=ints(E + 1), perm=ints(T * k),
                ws=runtime.empty_bytes(_lib.forge_moe_route_workspace_bytes(T, E, k)))


# ------------------------------------------------------------------- run ----

def run(state):
    return {"model": _run_model, "layer": _run_layer, "attention": _run_attention,
            "head": _run_head, "projection": _run_projection,
            "routing": _run_routing}[state["kind"]](state)


def _run_model(s):
    m = s["model"]
    loss = m.train_step(max_norm=1.0)
    f = m.flat
    return dict(loss=loss, grad={n: f.view(f.grad, n) for n in s["names"]}, master=f.master,
                param=f.param, m=f.m, v=f.v)


def _run_layer(s):
    ly = s["layer"]
    if s["moe"]:
        ly.aux.zero_()
    r = dict(out=s["out"], dx=s["dx"], grad=ly.g)
    if s["adamw"]:
        _lib.forge_adamw_advance(s["scalars"], s["step"], LR, BETA1, BETA2)
        ly.fwd(s["x"][0], s["out"][0])
        ly.bwd_adamw(s["x"][0], s["dy"][0], s["dx"][0], s["flat"], s["hp"], s["scalars"])
        f = s["flat"]
        r.update(master=f.master, param=f.param, m=f.m, v=f.v)
    else:
        for j, (x, dy, out, dx) in enumerate(zip(s["x"], s["dy"], s["out"], s["dx"])):
            ly.fwd(x, out)
            ly.bwd(x, dy, dx, overwrite=j == 0)
    if s["moe"]:
        r["aux"] = ly.aux
    return r


def _run_attention(s):
    _lib.forge_attention_fwd(s["cfg"], s["qkv"], s["o"], s["lse"])
    _lib.forge_attention_bwd(s["cfg"], s["qkv"], s["o"], s["lse"], s["do"], s["dqkv"], s["ws"])
    return dict(o=s["o"], lse=s["lse"], dqkv=s["dqkv"])


def _run_head(s):
    s["dg"].zero_()
    s["dw"].zero_()
    args = (s["x"], s["g"], s["w"], s["targets"], s["loss"], s["dx"], s["dg"], s["dw"], s["ws"])
    if s["chunk"]:
        _lib.forge_loss_fwd_bwd_chunked(s["cfg"], s["chunk"], *args)
    else:
        _lib.forge_loss_fwd_bwd(s["cfg"], *args)
    return dict(loss=s["loss"], dx=s["dx"], dg=s["dg"], dw=s["dw"])


def _run_projection(s):
    (T, k), n = s["x"].shape, s["w"].shape[0]
    kc, mc = _lib.GEMM_KC, _lib.GEMM_MC
    _lib.forge_gemm(kc, kc, _lib.EPI_STORE_BF16, s["x"], s["w"], s["y"], None, T, n, k, k, k, n)
    _lib.forge_gemm(kc, mc, _lib.EPI_STORE_BF16, s["dy"], s["w"], s["dx"], None, T, k, n, n, k, k)
    _lib.forge_gemm(mc, mc, _lib.EPI_STORE_F32, s["dy"], s["x"], s["dw"], None, n, k, T, n, k, k)
    return dict(y=s["y"], dx=s["dx"], dw=s["dw"])


def _run_routing(s):
    _lib.forge_moe_route(s["logits"], s["T"], s["E"], s["k"], s["idx"], s["gates"], s["probs"],
                         s["counts"], s["offsets"], s["perm"], s["ws"])
    return {n: s[n] for n in ("idx", "gates", "probs", "counts", "offsets", "perm")}


# ------------------------------------------------------------------ work ----

def _elements(shapes):
    return sum(math.prod(s) for s in shapes.values())


def _layer_work(c):
    """(bytes, flops) of a layer's forward and backward: products, attention
    over unmasked pairs; activations in and out, weights, gradients."""
    T, h, hq = c["batch"] * c["seq"], c["hidden"], c["n_heads"] * c["head_dim"]
    shapes = runtime.layer_shapes(c)
    n = _elements(shapes)
    used = n
    if c["n_experts"]:
        experts = math.prod(shapes["w_gate_up_e"]) + math.prod(shapes["w_down_e"])
        used = n - experts + experts * c["top_k"] / c["n_experts"]
    pairs = c["batch"] * c["seq"] * (c["seq"] + 1) / 2
    fwd_attention = 4 * pairs * hq
    flops = 6 * T * used + fwd_attention * (4 if c["recompute_attn"] else 3)
    return 2 * n + 4 * n + 8 * T * h, flops


def work(case):
    c, kind = case, case["kind"]
    if kind == "layer":
        b, f = _layer_work(c)
        n = _elements(runtime.layer_shapes(c))
        update = 26 * n if c["adamw"] else 0  # master, m, v read and written, param written
        return dict(bytes=c["micro"] * b + update, flops=c["micro"] * f)
    if kind == "model":
        T, h, V = c["batch"] * c["seq"], c["hidden"], c["vocab"]
        b, f = _layer_work(c)
        tables = V * h * (1 if c["tied"] else 2) + h
        n = c["n_layers"] * _elements(runtime.layer_shapes(c)) + tables
        return dict(bytes=36 * n + 8 * T + 8 * T * h, flops=c["n_layers"] * f + 6 * T * V * h)
    if kind == "attention":
        T, hq, hkv = c["batch"] * c["seq"], c["n_heads"] * c["head_dim"], c["n_kv_heads"] * c["head_dim"]
        pairs = c["batch"] * c["seq"] * (c["seq"] + 1) / 2
        return dict(bytes=2 * T * (2 * hq + 2 * (hq + 2 * hkv)) + 4 * c["n_heads"] * T,
                    flops=4 * pairs * hq * 3.5)
    if kind == "head":
        T, h, V = c["tokens"], c["hidden"], c["vocab"]
        return dict(bytes=4 * T * h + 6 * V * h + 4 * T, flops=6 * T * V * h)
    if kind == "projection":
        T, n, k = c["tokens"], c["n_out"], c["n_in"]
        return dict(bytes=4 * T * k + 4 * T * n + 6 * n * k, flops=6 * T * n * k)
    T, E, k = c["tokens"], c["n_experts"], c["top_k"]
    return dict(bytes=8 * T * E + 12 * T * k, flops=0)


def tolerance(case):
    """Relative errors, from what each kind shows against float64: bf16
    activations and gradients through a chain of layers (1.2e-2) or one layer
    (up to 9e-3), attention and the head (2.5e-3), one rounding of a product
    (1.7e-3), fp32 softmax (6e-8)."""
    return {"model": {"rel": 3e-2, "max": 0.5}, "layer": {"rel": 2.5e-2, "max": 0.5},
            "attention": {"rel": 1e-2, "max": 0.3}, "head": {"rel": 1e-2, "max": 0.3},
            "projection": {"rel": 7e-3, "max": 0.03}, "routing": {"rel": 1e-6, "max": 1e-5},
            }[case["kind"]]


# ----------------------------------------------------------------- exact ----

class _Attention64(torch.autograd.Function):
    """Causal grouped-query attention in float64, a head at a time (the score
    matrices are formed again in the backward)."""

    @staticmethod
    def scores(q, k):
        s = (q @ k.t()) / math.sqrt(q.shape[1])
        n = q.shape[0]
        return s.masked_fill_(torch.ones((n, n), dtype=torch.bool, device=DEV).triu_(1), -math.inf)

    @staticmethod
    def forward(ctx, q, k, v, batch):
        """q [T, nh, d], k and v [T, nkv, d] -> o [T, nh, d], lse [batch, nh, seq]."""
        T, nh, _ = q.shape
        S, grp = T // batch, nh // k.shape[1]
        o, lse = torch.empty_like(q), q.new_empty((batch, nh, S))
        for b in range(batch):
            r = slice(b * S, (b + 1) * S)
            for n in range(nh):
                s = _Attention64.scores(q[r, n], k[r, n // grp])
                lse[b, n] = torch.logsumexp(s, 1)
                o[r, n] = torch.exp(s - lse[b, n][:, None]) @ v[r, n // grp]
        ctx.save_for_backward(q, k, v, o, lse)
        ctx.mark_non_differentiable(lse)
        return o, lse

    @staticmethod
    def backward(ctx, do, _):
        q, k, v, o, lse = ctx.saved_tensors
        batch, nh, S = lse.shape
        grp, scale = nh // k.shape[1], 1.0 / math.sqrt(q.shape[2])
        dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
        for b in range(batch):
            r = slice(b * S, (b + 1) * S)
            for n in range(nh):
                m = n // grp
                p = torch.exp(_Attention64.scores(q[r, n], k[r, m]) - lse[b, n][:, None])
                dv[r, m] += p.t() @ do[r, n]
                p *= do[r, n] @ v[r, m].t() - (do[r, n] * o[r, n]).sum(1, keepdim=True)
                dq[r, n] = p @ k[r, m] * scale
                dk[r, m] += p.t() @ q[r, n] * scale
        return dq, dk, dv, None


def _rms64(x, g, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g


def _rope64(x, pos, base):
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * base ** (-torch.arange(half, device=DEV).double() / half)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)


def _ffn64(x, w_gate_up, w_down):
    g, u = (x @ w_gate_up.t()).chunk(2, 1)
    return (torch.nn.functional.silu(g) * u) @ w_down.t()


def _layer64(c, w, x, positions):
    """(out, aux) of one layer."""
    T, d, nh, nkv = c["batch"] * c["seq"], c["head_dim"], c["n_heads"], c["n_kv_heads"]
    pos = torch.arange(T, device=DEV) % c["seq"] if positions is None else positions
    scale = c["branch_scale"] or 1.0
    qkv = (_rms64(x, w["attn_norm"], c["rms_eps"]) @ w["w_qkv"].t()).view(T, nh + 2 * nkv, d)
    q, k, v = qkv.split([nh, nkv, nkv], 1)
    if c["qk_norm"]:
        q, k = _rms64(q, w["q_norm"], c["rms_eps"]), _rms64(k, w["k_norm"], c["rms_eps"])
    q, k = _rope64(q, pos, c["rope_base"]), _rope64(k, pos, c["rope_base"])
    o, _ = _Attention64.apply(q, k, v, c["batch"])
    h1 = x + scale * (o.reshape(T, nh * d) @ w["w_o"].t())
    b = _rms64(h1, w["ffn_norm"], c["rms_eps"])
    if not c["n_experts"]:
        return h1 + scale * _ffn64(b, w["w_gate_up"], w["w_down"]), None
    E, top = c["n_experts"], c["top_k"]
    logits = b @ w["w_router"].t()
    probs = logits.softmax(1)
    idx = logits.topk(top, dim=1).indices
    y = torch.zeros_like(h1)
    for e in range(E):
        rows = (idx == e).any(1).nonzero()[:, 0]
        y = y.index_add(0, rows, probs[rows, e][:, None]
                        * _ffn64(b[rows], w["w_gate_up_e"][e], w["w_down_e"][e]))
    if c["shared_ffn"]:
        y = y + _ffn64(b, w["w_gate_up_s"], w["w_down_s"])
    share = torch.bincount(idx.reshape(-1), minlength=E).double() / (T * top)
    return h1 + scale * y, c["aux_coef"] * E * (share * probs.mean(0)).sum()


def _adamw64(p, g, m, v, clip=1.0):
    """(master, m, v) after one more step of AdamW."""
    b1, b2 = float(np.float32(BETA1)), float(np.float32(BETA2))
    g = g * clip
    m, v = b1 * m.double() + (1 - b1) * g, b2 * v.double() + (1 - b2) * g.square()
    mh, vh = m / (1 - BETA1 ** (STEP + 1)), v / (1 - BETA2 ** (STEP + 1))
    return p - LR * (mh / (vh.sqrt() + ADAM_EPS) + WEIGHT_DECAY * p), m, v


def _leaf(t):
    return t.double().requires_grad_()


def _flat64(names, parts):
    """Tensors at the 64-element-aligned offsets of the flat buffers."""
    return torch.cat([torch.nn.functional.pad(parts[n].reshape(-1), (0, -parts[n].numel() % 64))
                      for n in names])


def exact(case, seed):
    """Every output with an error to measure. The loss and the load-balance
    loss are single numbers, whose distance from these is a matter of chance
    (a mean over all tokens of rounded values): None."""
    return {"model": _exact_model, "layer": _exact_layer, "attention": _exact_attention,
            "head": _exact_head, "projection": _exact_projection,
            "routing": _exact_routing}[case["kind"]](case, seed)


def _exact_layer(c, seed):
    i = _layer_inputs(c, seed)
    w = {n: _leaf(t) for n, t in i["w"].items()}
    r = dict(out=[], dx=[])
    for x, dy in zip(i["x"], i["dy"]):
        x = _leaf(x)
        out, aux = _layer64(c, w, x, i["positions"])
        ((out * dy.double()).sum() + (0.0 if aux is None else aux)).backward()
        r["out"].append(out.detach())
        r["dx"].append(x.grad)
    if c["n_experts"]:
        r["aux"] = None
    r["grad"] = {"d_" + n: t.grad for n, t in w.items()}
    if c["adamw"]:
        new = {n: _adamw64(t.detach().reshape(-1), t.grad.reshape(-1), *i["moments"][n])
               for n, t in w.items()}
        for k, name in enumerate(("master", "m", "v")):
            r[name] = _flat64(list(w), {n: t[k] for n, t in new.items()})
        r["param"] = r["master"]
    return r


def _exact_model(c, seed):
    i = _model_inputs(c, seed)
    p = {"embedding": _leaf(i["embedding"]), "final_norm": _leaf(i["final_norm"])}
    if not c["tied"]:
        p["w_lm"] = _leaf(i["w_lm"])
    layers = [{n: _leaf(t) for n, t in w.items()} for w in i["layers"]]
    for l, w in enumerate(layers):
        p.update({f"{l}.{n}": t for n, t in w.items()})
    x = p["embedding"][i["ids"].long()]
    for w in layers:
        x, _ = _layer64(c, w, x, None)
    z = _rms64(x, p["final_norm"], c["rms_eps"]) @ p["embedding" if c["tied"] else "w_lm"].t()
    loss = torch.nn.functional.cross_entropy(z, i["targets"].long())
    loss.backward()
    norm = math.sqrt(sum(float(t.grad.square().sum()) for t in p.values()))
    names, new = _model_names(c), {}
    for n in names:
        mom, var = _moments(i["moment_draw"], p[n].numel(), i["moment_scale"])
        new[n] = _adamw64(p[n].detach().reshape(-1), p[n].grad.reshape(-1), mom, var,
                          min(1.0, 1.0 / (norm + 1e-6)))
    r = dict(loss=None, grad={n: p[n].grad for n in names})
    for k, name in enumerate(("master", "m", "v")):
        r[name] = _flat64(names, {n: t[k] for n, t in new.items()})
    r["param"] = r["master"]
    return r


def _exact_attention(c, seed):
    qkv, do = _attention_inputs(c, seed)
    T, nh, nkv, d = c["batch"] * c["seq"], c["n_heads"], c["n_kv_heads"], c["head_dim"]
    x = _leaf(qkv)
    q, k, v = x.view(T, nh + 2 * nkv, d).split([nh, nkv, nkv], 1)
    o, lse = _Attention64.apply(q, k, v, c["batch"])
    o.backward(do.double().view(T, nh, d))
    return dict(o=o.detach().reshape(T, nh * d), lse=lse, dqkv=x.grad)


def _exact_head(c, seed):
    i = _head_inputs(c, seed)
    x, g, w = _leaf(i["x"]), _leaf(i["g"]), _leaf(i["w"])
    z = (_rms64(x, g, 1e-5) @ w.t()) * (c["logit_scale"] or 1.0)
    loss = torch.nn.functional.cross_entropy(z, i["targets"].long())
    loss.backward()
    return dict(loss=None, dx=x.grad, dg=g.grad, dw=w.grad)


def _exact_projection(c, seed):
    x, w, dy = (t.double() for t in _projection_inputs(c, seed))
    return dict(y=x @ w.t(), dx=dy @ w, dw=dy.t() @ x)


def _exact_routing(c, seed):
    """Probabilities and gates; the whole numbers have no error to measure."""
    logits = _Draw(seed).normal((c["tokens"], c["n_experts"]), 1.0)
    probs = logits.double().softmax(1)
    gates = probs.gather(1, logits.topk(c["top_k"], dim=1).indices)
    return dict(idx=None, gates=gates, probs=probs, counts=None, offsets=None, perm=None)
