"""Workloads of the W4A4 encoder linears that the performance of the library is judged by.

A case is a dict of plain values.  Three kinds of work, each through the public binding:

  layer    one BERT encoder layer, fp16 in and fp16 out (EncoderLayer): what serving calls per layer.
           Parts run as the built-in strategy table says; `fused_ln` lets FFN1 read the codes that
           LayerNorm 1 produced.
  linears  the four linears of an encoder layer, each from its own fp16 activations: token-wise
           quantize and the fused GEMM, calls marshalled once (Prepared...).  `form` is the
           arithmetic: "sym" (per-channel INT4, the layout the library prefers), "fp6" (the same in
           the FP6 operand layout), "asym" (per-channel, unsigned codes), "asym128" (unsigned codes,
           weight groups of 128), "int8" (the W8A8 sibling).
  chain    quantize once, then four linears that hand 4-bit codes to each other (requantizing
           epilogues), operands in `layout`.

Model sizes are BERT-base (768 / 3072) and BERT-large (1024 / 4096).
"""
import math

import torch

from paper_2301_12017_amd import binding as B
from paper_2301_12017_amd import synth
from paper_2301_12017_amd.workloads import ChainLayer, Layer, run_chain

FFN = {768: 3072, 1024: 4096}
SHAPES = ("qkv", "attn_out", "ffn1", "ffn2")
FORMS = ("sym", "fp6", "asym", "asym128", "int8")


def listed():
    return [
        # one short sentence, one ordinary one: interactive use at batch 1, where launches and latency count
        {"name": "layer_base_1x32", "kind": "layer", "hidden": 768, "batch": 1, "seq": 32, "fused_ln": False},
        {"name": "layer_base_1x128", "kind": "layer", "hidden": 768, "batch": 1, "seq": 128, "fused_ln": False},
        # a few requests of an odd length batched together
        {"name": "layer_base_5x93", "kind": "layer", "hidden": 768, "batch": 5, "seq": 93, "fused_ln": False},
        # longer documents on the larger model, nothing a multiple of anything
        {"name": "layer_large_9x371", "kind": "layer", "hidden": 1024, "batch": 9, "seq": 371, "fused_ln": False},
        # offline scoring: many ordinary sentences, and the longest sequences of the larger model
        {"name": "layer_base_128x128", "kind": "layer", "hidden": 768, "batch": 128, "seq": 128, "fused_ln": False},
        {"name": "layer_large_24x512", "kind": "layer", "hidden": 1024, "batch": 24, "seq": 512, "fused_ln": True},
        # the linears alone, for a program with an attention of its own: the throughput-oriented point of the paper
        {"name": "linears_large_12288", "kind": "linears", "hidden": 1024, "tokens": 12288, "form": "sym"},
        # the same layer kept in the FP6 operand layout, a ragged number of tokens
        {"name": "linears_large_fp6_8191", "kind": "linears", "hidden": 1024, "tokens": 8191, "form": "fp6"},
        # asymmetric activations with outlier channels, weights in groups of 128
        {"name": "linears_base_asym128_16384", "kind": "linears", "hidden": 768, "tokens": 16384, "form": "asym128"},
        # asymmetric codes for a small ragged batch
        {"name": "linears_base_asym_301", "kind": "linears", "hidden": 768, "tokens": 301, "form": "asym"},
        # layers that stay in eight bits
        {"name": "linears_large_int8_4096", "kind": "linears", "hidden": 1024, "tokens": 4096, "form": "int8"},
        # codes handed from layer to layer, no fp16 activation in between
        {"name": "chain_large_32768", "kind": "chain", "hidden": 1024, "tokens": 32768, "layout": "mfma"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    hidden = rng.choice((768, 1024))
    kind = rng.choice(("layer", "layer", "layer", "linears", "linears", "linears", "chain"))
    if kind == "layer":
        tokens, seq = _log_uniform(rng, 32, 12288), _log_uniform(rng, 16, 512)
        return {"kind": kind, "hidden": hidden, "batch": max(1, tokens // seq), "seq": seq, "fused_ln": rng.random() < 0.3}
    if kind == "linears":
        return {"kind": kind, "hidden": hidden, "tokens": _log_uniform(rng, 17, 16384), "form": rng.choice(FORMS)}
    layout = rng.choice(("mfma", "fp6"))        # (the FP6 layout has no rows of 3 * 768 codes)
    return {"kind": kind, "hidden": hidden if layout == "mfma" else 1024, "tokens": _log_uniform(rng, 500, 32768), "layout": layout}


def _dims(hidden):
    """{name: (N, K)} of the four linears."""
    f = FFN[hidden]
    return {"qkv": (3 * hidden, hidden), "attn_out": (hidden, hidden), "ffn1": (f, hidden), "ffn2": (hidden, f)}


class _Draws:
    """Normal fp16 tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def __call__(self, shape, std=1.0, mean=0.0):
        return (torch.randn(shape, generator=self.g, device="cuda") * std + mean).half()


def _act(name):
    return B.ACT_GELU if name == "ffn1" else B.ACT_NONE


def _prepare_layer(case, r):
    h, f, M = case["hidden"], FFN[case["hidden"]], case["batch"] * case["seq"]
    dims = _dims(h)
    args = []
    for name in SHAPES:         # the query and key weights give scores with a spread of about two, as trained ones do
        args += [r(dims[name], 0.05 if name == "qkv" else 0.02), r((dims[name][0],), 0.01)]
    for _ in range(2):
        args += [r((h,), 0.1, 1.0), r((h,), 0.1)]
    layer = B.EncoderLayer(case["batch"], case["seq"], h // 64, *args)
    strategy = B.strategy_lookup(M, h, f) | (B.STRATEGY_FUSED_LN if case["fused_ln"] else 0)
    return {"layer": layer, "strategy": strategy, "X": r((M, h)), "kind": "layer"}


def _prepare_linear(M, N, K, name, form, r):
    """The calls of one linear, in order, and its output."""
    X, W, bias = r((M, K)), r((N, K), 0.02), r((N,), 0.01)
    if form == "int8":
        wq, sw = B.quantize_rows8(W)
        q, s = torch.empty((M, K), dtype=torch.int8, device="cuda"), torch.empty((M,), device="cuda")
        lin = B.PreparedLinear8(q, s, wq, sw, bias, _act(name))
        return [B.PreparedQuantizeRows8(X, q, s), lin], lin.out
    mode, group = (B.ASYM, 128 if form == "asym128" else 0) if form.startswith("asym") else (B.SYM, 0)
    if mode == B.ASYM:          # a few hidden channels with a wide range, the same for every token
        X[:, torch.randperm(K, generator=r.g, device="cuda")[:8]] *= 20
    layout = B.LAYOUT_FP6 if form == "fp6" else B.preferred_layout(M, N, K, mode, group)
    Wq = B.quantize_weight(W, mode, group, layout)
    A = B.quantize_act(X, mode, group, layout=layout)
    lin = B.PreparedLinear(A, Wq, bias, _act(name))
    return [B.PreparedQuantizeAct(X, A), lin], lin.out[0]


def prepare(case, seed):
    r = _Draws(seed)
    if case["kind"] == "layer":
        return _prepare_layer(case, r)
    dims, M = _dims(case["hidden"]), case["tokens"]
    if case["kind"] == "linears":
        parts = [_prepare_linear(M, *dims[name], name, case["form"], r) for name in SHAPES]
        return {"kind": "linears", "calls": [c for calls, _ in parts for c in calls], "out": [out for _, out in parts]}
    layout = B.LAYOUT_FP6 if case["layout"] == "fp6" else B.LAYOUT_MFMA
    linears = []
    for name in SHAPES:
        N, K = dims[name]
        W = B.quantize_weight(r((N, K), 0.02), B.SYM, layout=layout)
        linears.append(Layer(synth.LinearSpec(name, M, N, K, name == "ffn1"), W, r((N,), 0.01), _act(name)))
    return {"kind": "chain", "layers": [ChainLayer(*linears)], "layout": layout, "X": r((M, case["hidden"]))}


def run(state):
    if state["kind"] == "layer":
        return state["layer"](state["X"], state["strategy"])
    if state["kind"] == "linears":
        for call in state["calls"]:
            call()
        return state["out"]
    out = run_chain(B.quantize_act(state["X"], B.SYM, layout=state["layout"]), state["layers"])
    if state["layout"] == B.LAYOUT_MFMA:        # (the layout's private code sums follow from the codes)
        return out.q, out.scale
    # whole panels of 64 tokens, and of the last one the rows that are tokens
    panels, rest = out.q.view(-1, out.K // 64, 64, 48), out.M % 64
    return (panels[:-1], panels[-1:, :, :rest], out.scale) if rest else (panels, out.scale)


def work(case):
    """Integer (and for the attention fp16) operations, and the bytes of inputs, weights and outputs, each once."""
    h = case["hidden"]
    M = case["batch"] * case["seq"] if case["kind"] == "layer" else case["tokens"]
    form = case.get("form", "fp6" if case.get("layout") == "fp6" else "sym")
    code = {"int8": 1.0, "fp6": 0.75}.get(form, 0.5)
    dims = _dims(h).values()
    weights = sum(n * k * code + 6 * n for n, k in dims)
    flops = sum(2.0 * M * n * k for n, k in dims)
    if case["kind"] == "layer":
        return {"bytes": weights + 4.0 * M * h, "flops": flops + 4.0 * M * case["seq"] * h}
    if case["kind"] == "linears":
        return {"bytes": weights + sum(2.0 * M * (n + k) for n, k in dims), "flops": flops}
    return {"bytes": weights + 2.0 * M * h + (code * h + 4.0) * M, "flops": flops}


def tolerance(case):
    """About four times what the same path shows with its floating-point parts evaluated in 64 bits."""
    if case["kind"] == "layer":
        # A last-bit difference of the attention or of LayerNorm 1 moves single 4-bit codes of the next part by one, and
        # where it moves a token's range or the codes behind it, a whole token a little: 3.4e-3, one element by 0.42.
        return {"rel": 1.2e-2, "max": 0.95}
    if case["kind"] == "linears":
        # Exact integer sums, fp32 dequantize, one rounding to fp16: 2.1e-4, one element 5e-4 (one step: 1e-3).  The large
        # terms of the unsigned mapping cancel: 3.9e-4, 2.1e-3.
        return {"rel": 1.6e-3, "max": 8e-3} if case["form"].startswith("asym") else {"rel": 8e-4, "max": 4e-3}
    # Exact up to GELU's last bits, which move 4e-6 of the third linear's codes by one and with them 3.6e-4 of the last
    # linear's; a scale by 4.6e-2 at most.
    return {"rel": 1.7e-3, "max": 0.18, "differ": 1.5e-3}
