"""bf16 attention backward at head sizes other than 64 and 128 where strips are too long for the workgroups to sum D = rowsum(dO * O) themselves: weights
stay float, and an infinity or a NaN stays out of the tokens that do not see it, in whole and in cut strips.  The same two properties that
test_gpu_attention_float_weights.py and test_gpu_attention_nonfinite.py ask of short strips, by their bounds; a sum over S
tokens is a chain of S / 16 matrix instructions, each of which adds a unit to the bound."""
import numpy as np
import pytest

import oracle
import test_gpu_attention_float_weights as weights

pytestmark = pytest.mark.gpu
CASES = [(8, 1025, None), (32, 1025, None), (40, 1025, None), (40, 1153, "17"), (80, 769, None), (104, 769, None), (104, 1025, "13")]


def _attention(pkg, torch, S, nl, dh, causal, qkv, d_o, cut):
    """o, dqkv, lse, and whether the row-dot kernel ran."""
    from torch.profiler import ProfilerActivity, profile
    dt, st = pkg.TPL_BF16, torch.cuda.current_stream()
    o, dqkv, ws = torch.empty_like(d_o), torch.empty_like(qkv), [None, None]
    lse, dsum = torch.empty(1, nl, S, device="cuda"), torch.empty(1, nl, S, device="cuda")
    if cut:
        ws = [torch.empty(max(pkg.tp_layer_attn_workspace_bytes(dt, 1, S, nl, dh, causal, bwd), 16), dtype=torch.uint8, device="cuda") for bwd in (False, True)]
    pkg.tp_layer_attn_fwd(dt, 1, S, nl, dh, causal, qkv, o, lse, ws=ws[0], stream=st)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        pkg.tp_layer_attn_bwd(dt, 1, S, nl, dh, causal, qkv, o, lse, d_o, dqkv, dsum, ws=ws[1], stream=st)
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "attn" in e.name]
    assert any("attn_dsum" in n for n in names) and any("combine" in n for n in names) == bool(cut), names
    return o, dqkv, lse


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,S,chunk", CASES)
def test_weights_stay_float(dh, S, chunk, causal, tune):
    import torch
    import paper_2111_05972_amd as pkg
    tune.set("attn_chunk", chunk)
    nl, dt, units = 2, pkg.TPL_BF16, (64 + S / 16) * 2.0 ** -24
    print(f"\n[attn] dh={dh} S={S} causal={causal} chunk={chunk}", flush=True)
    qkv, d_o = weights._draw(33, (S, 3 * nl * dh)), weights._draw(34, (S, nl * dh))
    o, dqkv, lse = _attention(pkg, torch, S, nl, dh, causal, pkg.to_device(qkv, dt), pkg.to_device(d_o, dt), chunk)
    heads = lambda x: x.astype(np.float64).reshape(1, S, nl, dh).transpose(0, 2, 1, 3)   # noqa: E731
    t = lambda x: x.transpose(0, 1, 3, 2)   # noqa: E731
    w, scale = nl * dh, 1.0 / np.sqrt(dh)
    Q, K, V = (heads(qkv[:, i * w:(i + 1) * w]) for i in range(3))
    dO, O_got = heads(d_o), heads(o.float().cpu().numpy())
    dq, dk, dv = (heads(dqkv[:, i * w:(i + 1) * w].float().cpu().numpy()) for i in range(3))
    O, P, LSE = oracle.attention_fwd(Q, K, V, causal)
    dS = P * (dO @ t(V) - (dO * O_got).sum(-1, keepdims=True))
    mag = P * (np.abs(dO) @ t(np.abs(V)) + (np.abs(dO) * np.abs(O_got)).sum(-1, keepdims=True))
    for name, g, ref, terms in (("o", O_got, O, P @ np.abs(V)), ("dq", dq, dS @ K * scale, mag @ np.abs(K) * scale),
                                ("dk", dk, t(dS) @ Q * scale, t(mag) @ np.abs(Q) * scale), ("dv", dv, t(P) @ dO, t(P) @ np.abs(dO))):
        over = np.abs(g - ref) - weights._half_ulp(ref, g) - units * terms
        assert (over <= 0).all(), (name, float((over > 0).mean()), float(over.max()))
    assert np.abs(lse.cpu().numpy() - LSE).max() <= units * np.abs(LSE).max()


def _reference(qkv, d_o, S, nl, dh, causal):
    """o, dqkv, lse over unmasked positions only, in float64."""
    w, scale = nl * dh, 1.0 / np.sqrt(dh)
    o, dqkv, lse = np.zeros((S, w)), np.zeros((S, 3 * w)), np.zeros((nl, S))
    for h in range(nl):
        Q, K, V = (qkv[:, i * w + h * dh:i * w + (h + 1) * dh].astype(np.float64) for i in range(3))
        dO, sl = d_o[:, h * dh:(h + 1) * dh].astype(np.float64), slice(h * dh, (h + 1) * dh)
        P, dS = np.zeros((S, S)), np.zeros((S, S))
        for i in range(S):
            n = i + 1 if causal else S
            s = K[:n] @ Q[i] * scale
            lse[h, i] = s.max() + np.log(np.exp(s - s.max()).sum())
            P[i, :n] = np.exp(s - lse[h, i])
            o[i, sl] = P[i, :n] @ V[:n]
            dS[i, :n] = P[i, :n] * (V[:n] @ dO[i] - dO[i] @ o[i, sl])
            dqkv[i, sl] = dS[i, :n] @ K[:n] * scale
        for j in range(S):
            first = j if causal else 0
            dqkv[j, w + h * dh:w + (h + 1) * dh] = dS[first:, j] @ Q[first:] * scale
            dqkv[j, 2 * w + h * dh:2 * w + (h + 1) * dh] = P[first:, j] @ dO[first:]
    return o, dqkv, lse


@pytest.mark.filterwarnings("ignore::RuntimeWarning")
@pytest.mark.parametrize("what,causal", [("q", True), ("k", True), ("v", True), ("do", True), ("v", False), ("do", False)])
@pytest.mark.parametrize("dh,S,chunk", [(32, 1025, None), (40, 1025, None), (40, 1153, "17"), (80, 769, None), (104, 1025, "13")])
def test_masked_tokens_stay_out(dh, S, chunk, what, causal, tune):
    import torch
    import paper_2111_05972_amd as pkg
    tune.set("attn_chunk", chunk)
    nl = 2
    for token, value in ((150, np.inf), (S - 3, np.nan)):
        print(f"\n[attn] dh={dh} S={S} chunk={chunk} causal={causal}: {value} in {what} of token {token}", flush=True)
        qkv, d_o = weights._draw(43, (S, 3 * nl * dh)).astype(np.float32), weights._draw(44, (S, nl * dh)).astype(np.float32)
        if what == "do":
            d_o[token, 3] = value
        else:
            qkv[token, "qkv".index(what) * nl * dh + 3] = value
        refs = _reference(qkv, d_o, S, nl, dh, causal)
        dev = lambda x: torch.from_numpy(x).to("cuda", torch.bfloat16)   # noqa: E731
        o, dqkv, lse = _attention(pkg, torch, S, nl, dh, causal, dev(qkv), dev(d_o), chunk)
        for name, got, ref in zip(("o", "dqkv", "lse"), (o, dqkv, lse[0]), refs):
            got, fin = got.float().cpu().numpy(), np.isfinite(ref)
            assert np.isfinite(got[fin]).all(), (name, int((~np.isfinite(got[fin])).sum()))
            assert not np.isfinite(got[~fin]).any(), name
            assert np.abs(got[fin] - ref[fin]).max() <= 2e-2 * max(1.0, np.abs(ref[fin]).max()), name
