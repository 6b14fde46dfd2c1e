"""GPU parity of forge_layer_fwd / forge_layer_bwd against the fp64 oracle.

Layer output and input gradient: relative Frobenius error <= 2e-2; every
fp32 weight gradient (accumulated into nonzero initial values) <= 3e-2.
"""
import numpy as np
import pytest

import forge_inputs as fi
from oracle import dense
from gpu_util import rel_fro, dev_bf16, host_f64, banner

pytestmark = pytest.mark.gpu

NAMES = ("attn_norm", "w_qkv", "w_o", "ffn_norm", "w_gate_up", "w_down")


def run_layer(cfg, seed=None, grad_init=0.0):
    import torch
    from paper_2609_13645_amd import runtime
    inp = fi.layer_inputs(cfg, seed)
    layer = runtime.Layer(cfg, inp["weights"])
    for t in layer.g.values():
        t.fill_(grad_init)
    x = dev_bf16(inp["x"])
    dy = dev_bf16(inp["dy"])
    out = torch.empty_like(x)
    dx = torch.empty_like(x)
    layer.fwd(x, out)
    layer.bwd(x, dy, dx)
    torch.cuda.synchronize()
    got = {"out": host_f64(out), "dx": host_f64(dx)}
    for n in NAMES:
        got[n] = host_f64(layer.g["d_" + n]) - grad_init
    W = {k: fi.bf16_bits_to_f64(v) for k, v in inp["weights"].items()}
    ref_out, cache = dense.layer_fwd(fi.bf16_bits_to_f64(inp["x"]), W, cfg)
    ref_dx, ref_g = dense.layer_bwd(cache, W, cfg, fi.bf16_bits_to_f64(inp["dy"]))
    ref = {"out": ref_out, "dx": ref_dx}
    ref.update(ref_g)
    return got, ref


def check(got, ref):
    errs = {k: rel_fro(got[k], ref[k]) for k in ref}
    banner(f"  errors {({k: f'{v:.2e}' for k, v in errs.items()})}")
    assert errs["out"] <= 2e-2 and errs["dx"] <= 2e-2
    for n in NAMES:
        assert errs[n] <= 3e-2, n
    for k, v in got.items():
        assert np.all(np.isfinite(v)), k


def test_layer_tiny():
    cfg = fi.config("tiny")
    banner(f"layer tiny T={fi.tokens(cfg)}")
    check(*run_layer(cfg, grad_init=0.5))


def test_layer_tiny_ragged_two_rows():
    cfg = fi.config("tiny", batch=2, seq=77)
    banner("layer tiny batch 2 seq 77")
    check(*run_layer(cfg, seed=11))


def test_layer_8b_geometry_short_seq():
    # the 8B-shape layer (h 4096, 32/8 heads of 128, f 14336) at 320 tokens:
    # several GEMM tiles plus a ragged tail, attention tiles 128 + ragged
    cfg = fi.config("llama8b_layer", seq=320)
    banner("layer llama8b geometry seq 320")
    check(*run_layer(cfg, seed=21))


@pytest.mark.parametrize("name,over,seed", [
    ("tiny", dict(batch=2, seq=77), 13),
    ("tiny", dict(seq=160, head_dim=128, n_heads=2, n_kv_heads=1), 5),
    ("llama8b_layer", dict(seq=320), 22),
])
def test_layer_recompute_attention_vs_oracle(name, over, seed):
    # attention recomputed in the backward (O and LSE not kept, Sec. 3.3
    # recompute policies): the whole layer backward against the oracle
    cfg = fi.config(name, recompute_attn=1, **over)
    banner(f"layer recompute_attn {name} {over}")
    check(*run_layer(cfg, seed=seed))


def test_layer_bwd_d_in_aliasing_d_out():
    """d_in may be the very buffer of d_out: with the side streams on (T x h
    >= 2^20) the result must equal the one with separate buffers, bit for
    bit, whatever the weight-gradient stream still reads."""
    import torch
    from paper_2609_13645_amd import runtime
    cfg = fi.config("llama8b_layer", seq=320)
    assert runtime.uses_side_streams(cfg)
    banner("layer backward with d_in == d_out (side streams)")
    inp = fi.layer_inputs(cfg, seed=23)
    res = []
    for alias in (False, True):
        layer = runtime.Layer(cfg, inp["weights"])
        x, dy = dev_bf16(inp["x"]), dev_bf16(inp["dy"])
        out = torch.empty_like(x)
        layer.fwd(x, out)
        dx = dy if alias else torch.empty_like(x)
        layer.bwd(x, dy, dx, overwrite=True)
        torch.cuda.synchronize()
        res.append([host_f64(dx)] + [host_f64(layer.g["d_" + n]) for n in NAMES])
    for n, a, b in zip(("dx",) + NAMES, *res):
        assert np.array_equal(a, b), n


def test_layer_recompute_matches_stored():
    import torch
    from paper_2609_13645_amd import runtime
    cfg = fi.config("tiny", seq=160, head_dim=128, n_heads=2, n_kv_heads=1)
    banner("layer recompute vs stored attention")
    inp = fi.layer_inputs(cfg, seed=5)
    res = []
    for rec in (0, 1):
        c = dict(cfg, recompute_attn=rec)
        layer = runtime.Layer(c, inp["weights"])
        x, dy = dev_bf16(inp["x"]), dev_bf16(inp["dy"])
        out, dx = torch.empty_like(x), torch.empty_like(x)
        layer.fwd(x, out)
        layer.bwd(x, dy, dx)
        torch.cuda.synchronize()
        res.append([host_f64(out), host_f64(dx)] + [host_f64(layer.g["d_" + n]) for n in NAMES])
    for a, b in zip(*res):
        assert np.array_equal(a, b)


def test_layer_is_deterministic():
    cfg = fi.config("tiny", seq=200)
    banner("layer determinism")
    a, _ = run_layer(cfg, seed=3)
    b, _ = run_layer(cfg, seed=3)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("which", ["dense", "moe"])
def test_overwrite_grads_equal_accumulate_into_zeros(which):
    """grads.overwrite writes every weight gradient: bitwise the values that
    accumulating into zeroed buffers gives, whatever the buffers held."""
    import torch
    from paper_2609_13645_amd import runtime
    if which == "dense":
        cfg = fi.config("tiny", batch=2, seq=72, seed=17)
    else:
        cfg = fi.config("tiny", batch=1, seq=2048, ffn=0, n_experts=16, top_k=2,
                        expert_ffn=64, aux_coef=0.05, seed=61)
    banner(f"overwrite vs accumulate ({which})")
    inp = fi.layer_inputs(cfg)
    layer = runtime.Layer(cfg, inp["weights"])
    x, dy = dev_bf16(inp["x"]), dev_bf16(inp["dy"])
    out, dx = torch.empty_like(x), torch.empty_like(x)
    layer.fwd(x, out)
    layer.zero_grads()
    layer.bwd(x, dy, dx)
    torch.cuda.synchronize()
    acc = {k: v.clone() for k, v in layer.g.items()}
    for v in layer.g.values():
        v.fill_(float("nan"))
    layer.bwd(x, dy, dx, overwrite=True)
    torch.cuda.synchronize()
    for k, v in layer.g.items():
        assert torch.equal(v, acc[k]), k


@pytest.mark.parametrize("over", [
    # few tokens, wide heads and FFN: the O and down forward products and the
    # QKV and gate/up data gradients split (K 4096 to 8208)
    dict(batch=1, seq=72, hidden=512, n_heads=32, n_kv_heads=8, head_dim=128, ffn=4104),
    # many tokens, narrow layer: all four weight gradients split (K = 2064)
    dict(batch=2, seq=1032, hidden=264, n_heads=4, n_kv_heads=1, head_dim=64, ffn=520),
])
def test_layer_split_reductions(over):
    """Layers whose products split their reduction over workgroups, against
    the oracle; and a forward without a workspace, whose products do not
    split: the same up to the order of the fp32 sums (one bf16 rounding of
    the output either way)."""
    import torch
    from paper_2609_13645_amd import _lib, runtime
    cfg = fi.config("tiny", **over)
    banner(f"layer split reductions {over}")
    check(*run_layer(cfg, seed=71))
    inp = fi.layer_inputs(cfg, 71)
    layer = runtime.Layer(cfg, inp["weights"])
    x = runtime.to_device_bf16(inp["x"])
    a, b = torch.empty_like(x), torch.empty_like(x)
    layer.fwd(x, a)
    _lib.forge_layer_fwd(layer.c, layer.weights, x, b, layer.saved, None)
    torch.cuda.synchronize()
    assert rel_fro(host_f64(a), host_f64(b)) <= 4e-3
