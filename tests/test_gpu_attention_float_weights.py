"""GPU: bf16 attention at head sizes other than 64 and 128 multiplies float probabilities and float dS (not their bf16
roundings) with V, dO, K and Q.  Every element of the result is then the correctly rounded float64 one up to float
arithmetic:

    |got - ref| <= half a bf16 ulp + 64 * 2^-24 * (sum of the magnitudes of the element's terms)

with 64 units for the chain of a weight (dot product of up to 128 terms, exponent argument of up to 20, row sum).  A weight
rounded to bf16 is off by up to 2^-9 of itself, 500 times that bound."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu
UNITS = 64 * 2.0 ** -24


def _draw(seed, shape):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), 1.0), "bf16").reshape(shape)


def _half_ulp(ref, got):
    big = np.maximum(np.maximum(np.abs(ref), np.abs(got)), 2.0 ** -120)
    return 2.0 ** (np.floor(np.log2(big)) - 8)


@pytest.mark.parametrize("chunk", [None, "1"])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh", [8, 40, 80, 96, 104, 120])
def test_weights_stay_float(dh, causal, chunk, tune):
    import torch
    import paper_2111_05972_amd as pkg
    tune.set("attn_chunk", chunk)
    B, S, nl, dt, st = 1, 200, 2, pkg.TPL_BF16, torch.cuda.current_stream()
    print(f"\n[attn] float weights dh={dh} causal={causal} chunk={chunk}", flush=True)
    qkv, d_o = _draw(31, (B * S, 3 * nl * dh)), _draw(32, (B * S, nl * dh))
    qkv_d, d_o_d = pkg.to_device(qkv, dt), pkg.to_device(d_o, dt)
    o_d, dqkv = torch.empty_like(d_o_d), torch.empty_like(qkv_d)
    lse_d, dsum = torch.empty(B, nl, S, device="cuda"), torch.empty(B, nl, S, device="cuda")
    ws = [None, None]
    if chunk:
        ws = [torch.empty(max(pkg.tp_layer_attn_workspace_bytes(dt, B, S, nl, dh, causal, bwd), 16), dtype=torch.uint8, device="cuda")
              for bwd in (False, True)]
    pkg.tp_layer_attn_fwd(dt, B, S, nl, dh, causal, qkv_d, o_d, lse_d, ws=ws[0], stream=st)
    pkg.tp_layer_attn_bwd(dt, B, S, nl, dh, causal, qkv_d, o_d, lse_d, d_o_d, dqkv, dsum, ws=ws[1], stream=st)
    torch.cuda.synchronize()
    heads = lambda x: x.astype(np.float64).reshape(B, S, nl, dh).transpose(0, 2, 1, 3)   # noqa: E731
    w = nl * dh
    Q, K, V = (heads(qkv[:, i * w:(i + 1) * w]) for i in range(3))
    dO, O_got = heads(d_o), heads(o_d.float().cpu().numpy())
    got = [heads(dqkv[:, i * w:(i + 1) * w].float().cpu().numpy()) for i in range(3)]
    O, P, LSE = oracle.attention_fwd(Q, K, V, causal)
    t = lambda x: x.transpose(0, 1, 3, 2)   # noqa: E731
    D = (dO * O_got).sum(-1, keepdims=True)                       # the backward pass reads the rounded O
    dS, mag = P * (dO @ t(V) - D), P * (np.abs(dO) @ t(np.abs(V)) + (np.abs(dO) * np.abs(O_got)).sum(-1, keepdims=True))
    scale = 1.0 / np.sqrt(dh)
    for name, g, ref, terms in (("o", O_got, O, P @ np.abs(V)),
                                ("dq", got[0], dS @ K * scale, mag @ np.abs(K) * scale),
                                ("dk", got[1], t(dS) @ Q * scale, t(mag) @ np.abs(Q) * scale),
                                ("dv", got[2], t(P) @ dO, t(P) @ np.abs(dO))):
        over = np.abs(g - ref) - _half_ulp(ref, g) - UNITS * terms
        assert (over <= 0).all(), (name, float((over > 0).mean()), float(over.max()))
    assert np.abs(lse_d.cpu().numpy() - LSE).max() <= UNITS * np.abs(LSE).max()
