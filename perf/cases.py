"""The measured workloads: what a program built on this package has it do, through its public entry points.

Kinds of case:
  step    training step of one rank's layer shard: TpLayer.forward, then TpLayer.backward
  eval    forward only (evaluation, or the prefill of a short prompt)
  ckpt    training step with activation checkpointing: forward, then the backward that recomputes
  attn    softmax attention alone, forward and backward (tp_layer_attn_fwd, tp_layer_attn_bwd)
  ln      residual + LayerNorm alone, forward and backward (tp_layer_ln_fwd, tp_layer_ln_bwd)
  memopt  one rank's local compute of a training step in the memory-optimised distribution (MemOptRank)

Sizes are those of the named configurations of synthetic/configs.py, of bench.py and of the tests, or generic ones of
the same ranges.  Tensors are drawn as there: activations and upstream gradients N(0, 1), weights and biases
N(0, sigma_w) with sigma_w = 0.006 for the widest layers and 0.02 otherwise.
"""
import math

import torch

import paper_2111_05972_amd as pkg
from paper_2111_05972_amd.memopt import PARAM_SHAPES, MemOptRank

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
_TPL = {"f32": pkg.TPL_F32, "bf16": pkg.TPL_BF16}


def _layer(name, kind, dtype, hidden, heads, head_dim, tp, rank, seq, batch, causal, epilogue, chains):
    """chains: the two blocks of a pass as two chains (TPL_SIDE_STREAM), or every kernel on the caller's stream."""
    case = {"kind": kind, "dtype": dtype, "hidden": hidden, "heads": heads, "head_dim": head_dim,
            "intermediate": 4 * hidden, "tp": tp, "rank": rank, "seq": seq, "batch": batch, "causal": causal,
            "epilogue": epilogue, "chains": chains}
    return {"name": name, **case} if name else case


def listed():
    return [
        # the smallest shard anybody trains: bring-up and parity in float, one launch after another (tiny GPT, TP 2)
        _layer("step-tiny-f32", "step", "f32", 256, 4, 64, 2, 0, 128, 2, True, True, False),
        # float at a real width: a reference run of an encoder layer without bf16
        _layer("step-encoder-f32", "step", "f32", 1024, 16, 64, 4, 0, 512, 4, False, True, False),
        # encoder layers at sequence length 512, the short GEMMs of narrow shards (BERT-large TP 4, RoBERTa-large TP 2)
        _layer("step-bert-large-tp4", "step", "bf16", 1024, 16, 64, 4, 1, 512, 8, False, False, False),
        _layer("step-roberta-large-tp2", "step", "bf16", 1024, 16, 64, 2, 0, 512, 16, False, True, True),
        # decoder layers at sequence length 2048 (GPT-3 13B TP 4; GPT-3 175B TP 8 is the headline configuration)
        _layer("step-gpt3-13b-tp4", "step", "bf16", 5120, 40, 128, 4, 0, 2048, 2, True, True, True),
        _layer("step-gpt3-175b-tp8", "step", "bf16", 12288, 96, 128, 8, 3, 2048, 1, True, False, True),
        # sizes that divide by nothing: head size 80, an odd sequence length, three sequences in the micro-batch
        _layer("step-ragged", "step", "bf16", 2560, 32, 80, 4, 2, 1001, 3, True, True, True),
        # forward only, few tokens against the widest weights: bound by reading the weights once
        _layer("eval-short-175b-tp8", "eval", "bf16", 12288, 96, 128, 8, 0, 100, 1, True, True, False),
        # activations recomputed in backward (the 10B encoder shard)
        _layer("ckpt-roberta-10b-tp4", "ckpt", "bf16", 4096, 32, 128, 4, 0, 512, 8, False, True, True),
        # attention alone on a long causal sequence, with the workspace the library asks for
        {"name": "attn-long-causal", "kind": "attn", "dtype": "bf16", "batch": 1, "seq": 8192, "heads": 12, "head_dim": 128,
         "causal": True},
        # residual + LayerNorm around the widest shard
        {"name": "ln-2048x12288", "kind": "ln", "dtype": "bf16", "tokens": 2048, "hidden": 12288},
        # the other distribution: inputs split over channels, so K is short in forward and very long in the data gradients
        {"name": "memopt-13b-tp4", "kind": "memopt", "dtype": "bf16", "hidden": 5120, "heads": 40, "tp": 4, "seq": 2048,
         "batch": 1, "causal": True},
    ]


# What a drawn case may cost, in flops of one pass: no more than the widest listed step in bf16, and in float no more
# than a few of the listed encoder steps.
_MOST_FLOPS = {"bf16": 2.0e12, "f32": 2.0e11}


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_layer(rng, kind):
    dtype = "bf16" if kind == "memopt" or rng.random() < 0.75 else "f32"
    while True:
        head_dim = rng.choice([64, 64, 64, 128, 128, 128, 32, 80, 96, 104] if kind != "memopt" else [64, 128])
        tp = rng.choice([1, 2, 4, 8])
        local = max(1, round(_log_uniform(rng, 256, 12288 if dtype == "bf16" else 2048) / (head_dim * tp)))
        heads, hidden = local * tp, local * tp * head_dim
        if kind == "eval":
            seq, batch = round(_log_uniform(rng, 1, 512)), rng.choice([1, 1, 2, 4])
        else:
            seq, batch = round(_log_uniform(rng, 64, 4096)), round(_log_uniform(rng, 1, 16))
        case = _layer(None, kind, dtype, hidden, heads, head_dim, tp, rng.randrange(tp), seq, batch, rng.random() < 0.6,
                      rng.random() < 0.5, rng.random() < 0.6)
        if 256 <= hidden <= 12288 and seq * batch <= 16384 and work(case)["flops"] <= _MOST_FLOPS[dtype]:
            if kind == "memopt":
                return {k: case[k] for k in ("kind", "dtype", "hidden", "heads", "tp", "seq", "batch", "causal")}
            return case


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["eval", "ckpt", "attn", "attn", "ln", "ln", "memopt"])
    if kind == "ln":
        hidden = 8 * round(_log_uniform(rng, 256, 16384) / 8)
        tokens = round(_log_uniform(rng, 64, min(16384, 4.0e7 / hidden)))
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "f32"]), "tokens": tokens, "hidden": hidden}
    if kind == "attn":
        while True:
            case = {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"]), "batch": round(_log_uniform(rng, 1, 16)),
                    "seq": round(_log_uniform(rng, 64, 8192)), "heads": round(_log_uniform(rng, 1, 24)),
                    "head_dim": rng.choice([64, 64, 128, 128, 80]), "causal": rng.random() < 0.6}
            if work(case)["flops"] <= (6.0e11 if case["dtype"] == "bf16" else 3.0e10):
                return case
    return _draw_layer(rng, kind)


class _Random:
    """Seeded normal tensors on the GPU."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dtype = _TORCH[dtype]

    def __call__(self, *shape, sigma=1.0, mean=0.0, dtype=None):
        t = torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32)
        return t.mul_(sigma).add_(mean).to(dtype or self.dtype)


def _sigma_w(hidden):
    return 0.006 if hidden >= 8192 else 0.02


def prepare(case, seed):
    rnd = _Random(seed, case["dtype"])
    return {"attn": _prepare_attn, "ln": _prepare_ln, "memopt": _prepare_memopt}.get(case["kind"], _prepare_layer)(case, rnd)


def _prepare_layer(case, rnd):
    layer = pkg.TpLayer(case["hidden"], case["heads"], case["tp"], case["rank"], case["seq"], case["batch"],
                        _TPL[case["dtype"]], case["causal"], case["epilogue"], case["head_dim"], case["intermediate"],
                        side_stream=case["chains"])
    s = {"case": case, "layer": layer,
         "params": {k: rnd(*shape, sigma=_sigma_w(case["hidden"])) for k, shape in layer.param_shapes().items()},
         "x_attn": rnd(layer.M, layer.H), "x_mlp": rnd(layer.M, layer.H), "y": layer.empty_outputs()}
    if case["kind"] != "eval":
        s.update(dy_attn=rnd(layer.M, layer.H), dy_mlp=rnd(layer.M, layer.H), grads=layer.empty_grads(),
                 dx=layer.empty_outputs())
    if case["kind"] == "ckpt":
        s["ws"] = torch.empty(pkg.tp_layer_workspace_bytes_recompute(layer.desc), dtype=torch.uint8, device="cuda")
    return s


def _prepare_attn(case, rnd):
    dt, B, S, nl, dh, causal = (_TPL[case["dtype"]], case["batch"], case["seq"], case["heads"], case["head_dim"], case["causal"])
    qkv, d_o = rnd(B * S, 3 * nl * dh), rnd(B * S, nl * dh)
    nbytes = max(pkg.tp_layer_attn_workspace_bytes(dt, B, S, nl, dh, causal, bwd) for bwd in (False, True))
    return {"case": case, "args": (dt, B, S, nl, dh, causal), "qkv": qkv, "d_o": d_o, "o": torch.empty_like(d_o),
            "lse": torch.empty(B, nl, S, dtype=torch.float32, device="cuda"), "dqkv": torch.empty_like(qkv),
            "dsum": torch.empty(B, nl, S, dtype=torch.float32, device="cuda"),
            "ws": torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None}


def _prepare_ln(case, rnd):
    M, H = case["tokens"], case["hidden"]
    a, b, dy = rnd(M, H, mean=0.5), rnd(M, H), rnd(M, H)
    gamma, beta = rnd(H, sigma=0.2, mean=1.0), rnd(H, sigma=0.2)
    like = torch.empty_like
    return {"case": case, "a": a, "b": b, "dy": dy, "gamma": gamma, "beta": beta, "z": like(a), "y": like(a), "dz": like(a),
            "mean": torch.empty(M, dtype=torch.float32, device="cuda"), "rstd": torch.empty(M, dtype=torch.float32, device="cuda"),
            "dgamma": like(gamma), "dbeta": like(beta),
            "ws": torch.empty(pkg.tp_layer_ln_workspace_bytes(M, H), dtype=torch.uint8, device="cuda")}


def _prepare_memopt(case, rnd):
    H, I, T = case["hidden"], 4 * case["hidden"], case["tp"]
    rank = MemOptRank(H, case["heads"], I, T, case["seq"], case["batch"], _TPL[case["dtype"]], case["causal"])
    M, sw = rank.M, _sigma_w(H)
    params = {}
    for k, shape in PARAM_SHAPES(H, rank.Hs, rank.Hl, I, rank.Il).items():
        norm = k in ("g1", "b1", "g2", "b2")
        params[k] = rnd(*shape, sigma=0.1 if norm else sw, mean=1.0 if k in ("g1", "g2") else 0.0)
    # what the collectives would deliver: reduce-scattered slices, all-gathered gradients, all-reduced moments and sums
    given = {k: rnd(M, n) for k, n in (("x", rank.Hs), ("qkv_in", 3 * rank.Hl), ("o_in", rank.Hs), ("u_in", rank.Il),
                                       ("d_in", rank.Hs), ("dy2", rank.Hs), ("dy2_full", H), ("du_full", I),
                                       ("dy1_full", H), ("dqkv_full", 3 * H))}
    f32 = torch.float32
    for k, var in (("m1", 1.0), ("m2", 2.0)):
        given[k] = torch.stack([rnd(M, sigma=math.sqrt(H), dtype=f32), torch.full((M,), var * H, device="cuda")], 1).contiguous()
    for k in ("s1", "s2"):
        given[k] = rnd(M, 2, sigma=10.0, dtype=f32)
    return {"case": case, "rank": rank, "params": params, "in": given}


def run(s):
    kind = s["case"]["kind"]
    return {"attn": _run_attn, "ln": _run_ln, "memopt": _run_memopt}.get(kind, _run_layer)(s)


def _run_layer(s):
    layer, kind = s["layer"], s["case"]["kind"]
    y_attn, y_mlp = layer.forward(s["params"], s["x_attn"], s["x_mlp"], *s["y"])
    out = {"y_attn": y_attn, "y_mlp": y_mlp}
    if kind == "eval":
        return out
    dx_attn, dx_mlp = s["dx"]
    if kind == "step":
        layer.backward(s["params"], s["x_attn"], s["x_mlp"], s["dy_attn"], s["dy_mlp"], s["grads"], dx_attn, dx_mlp)
    else:
        pkg.tp_layer_bwd_recompute(layer.desc, s["params"], s["x_attn"], s["x_mlp"], s["dy_attn"], s["dy_mlp"], s["grads"],
                                   dx_attn, dx_mlp, s["ws"], stream=torch.cuda.current_stream())
    # without the row epilogue the biases of the row-split linears belong to another rank: their gradients are not written
    grads = {k: g for k, g in s["grads"].items() if s["case"]["epilogue"] or k not in ("db_o", "db_dn")}
    return {**out, "dx_attn": dx_attn, "dx_mlp": dx_mlp, **grads}


def _run_attn(s):
    stream = torch.cuda.current_stream()
    pkg.tp_layer_attn_fwd(*s["args"], s["qkv"], s["o"], s["lse"], ws=s["ws"], stream=stream)
    pkg.tp_layer_attn_bwd(*s["args"], s["qkv"], s["o"], s["lse"], s["d_o"], s["dqkv"], s["dsum"], ws=s["ws"], stream=stream)
    return {"o": s["o"], "lse": s["lse"], "dqkv": s["dqkv"]}


def _run_ln(s):
    dt, M, H, stream = _TPL[s["case"]["dtype"]], s["case"]["tokens"], s["case"]["hidden"], torch.cuda.current_stream()
    pkg.tp_layer_ln_fwd(dt, M, H, s["a"], s["b"], s["gamma"], s["beta"], 1e-5, s["z"], s["y"], s["mean"], s["rstd"], stream=stream)
    pkg.tp_layer_ln_bwd(dt, M, H, s["dy"], s["z"], s["mean"], s["rstd"], s["gamma"], s["dz"], s["dgamma"], s["dbeta"], s["ws"],
                        stream=stream)
    return {k: s[k] for k in ("z", "y", "mean", "rstd", "dz", "dgamma", "dbeta")}


def _run_memopt(s):
    rank, p, x = s["rank"], s["params"], s["in"]
    rank.f0_moments(p, x["x"])
    rank.f1_qkv_partial(x["m1"])
    rank.f2_attn_partial(x["qkv_in"])
    rank.f3_moments(x["o_in"])
    rank.f4_up_partial(x["m2"])
    part = rank.f5_down_partial(x["u_in"])
    y2 = rank.f6_finish(x["d_in"])
    rank.b0_start(x["dy2"])
    du = rank.b1_down(x["dy2_full"])
    rank.b2_up(x["du_full"])
    dy1 = rank.b3_ln2(x["s2"])
    dqkv = rank.b4_attn(x["dy1_full"])
    rank.b5_qkv(x["dqkv_full"])
    dx = rank.b6_ln1(x["s1"])
    return {"down_partial": part, "y2": y2, "du": du, "dy1": dy1, "dqkv": dqkv, "dx": dx, **rank.grads}


def _attn_flops(B, S, nl, dh, causal):
    """Forward: two products over the query-key pairs that the mask leaves; backward: twice that."""
    return 4.0 * B * nl * (S * (S + 1) / 2 if causal else float(S) * S) * dh


def work(case):
    size = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "ln":      # a, b, dy read; z, y, dz written (z need not be read back)
        n = case["tokens"] * case["hidden"]
        return {"bytes": 6.0 * n * size, "flops": 20.0 * n}
    if case["kind"] == "attn":    # qkv, dO read; O, dqkv, LSE written
        n = case["batch"] * case["seq"] * case["heads"]
        return {"bytes": 8.0 * n * case["head_dim"] * size + 4.0 * n,
                "flops": 3.0 * _attn_flops(case["batch"], case["seq"], case["heads"], case["head_dim"], case["causal"])}
    H, T, M = case["hidden"], case["tp"], case["seq"] * case["batch"]
    I = case.get("intermediate", 4 * H)
    Hl, Il, nl = H // T, I // T, case["heads"] // T
    params = H * (4.0 * Hl + 2.0 * Il)
    fwd = 2.0 * M * params + _attn_flops(case["batch"], case["seq"], nl, H // case["heads"], case["causal"])
    if case["kind"] == "eval":    # weights and both inputs read, both outputs written
        return {"bytes": (params + 4.0 * M * H) * size, "flops": fwd}
    if case["kind"] == "memopt":  # weights and what the collectives deliver read; weight gradients and what they collect written
        given = M * (4.0 * Hl + 3.0 * Hl + Il + 2.0 * H + I + 3.0 * H)
        sent = M * (3.0 * H + H + I + H + Hl + Il + Hl + 3.0 * Hl + Hl)
        return {"bytes": (2.0 * params + given + sent) * size, "flops": 3.0 * fwd}
    # weights, two inputs, two upstream gradients read; weight gradients, two outputs, two input gradients written
    recomputed = 2.0 * M * H * (3.0 * Hl + Il) + (fwd - 2.0 * M * params) if case["kind"] == "ckpt" else 0.0
    return {"bytes": (2.0 * params + 8.0 * M * H) * size, "flops": 3.0 * fwd + recomputed}


def tolerance(case):
    # Two-norm of the difference over the two-norm of the result, the worst output of a case.  Against the same pass in
    # 64 bits on the device: at most 1.2e-6 in float and 5.7e-3 in bf16 over the listed cases (the weight gradients
    # behind a long softmax: bf16 rounding of QKV, O, dO and dQKV), 6.8e-3 over drawn ones; stated with a margin.
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 2e-2}
