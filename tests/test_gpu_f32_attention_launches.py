"""Float attention backward on either side of the line between one launch that works D out by itself (at most a workgroup of 32
rows per compute unit, dQ and dK/dV together) and D in a launch before: dQ and dK/dV together at head sizes up to 64, dQ first
beyond.  Ragged rows, odd head sizes; against the oracle's definitions, and twice over bit-identical."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,S,nl,dh", [(8, 32, 16, 64), (43, 32, 3, 32), (2, 61, 32, 128), (5, 33, 16, 128), (1, 97, 2, 96), (13, 70, 4, 96), (3, 95, 29, 36),
                                       (17, 100, 5, 4), (2, 290, 13, 60)])
def test_one_launch_and_two(B, S, nl, dh, causal):
    import torch
    import paper_2111_05972_amd as pkg
    print(f"\n[attn f32] {B} {S} {nl} {dh} causal={causal}", flush=True)
    dt = pkg.TPL_F32
    qkv, d_o = synthetic.normal(41, B * S * 3 * nl * dh, 1.0), synthetic.normal(42, B * S * nl * dh, 1.0)
    qkv, d_o = (synthetic.quantize(v, "f32") for v in (qkv, d_o))
    t = qkv.reshape(B, S, 3, nl, dh).astype(np.float64)
    Q, K, V = (t[:, :, i].transpose(0, 2, 1, 3) for i in range(3))
    O, P, _ = oracle.attention_fwd(Q, K, V, causal)
    grads = oracle.attention_bwd(Q, K, V, P, d_o.reshape(B, S, nl, dh).transpose(0, 2, 1, 3).astype(np.float64))
    ref = np.stack([a.transpose(0, 2, 1, 3) for a in grads], axis=2).reshape(B * S, 3, nl * dh)
    x, g = pkg.to_device(qkv.reshape(B * S, -1), dt), pkg.to_device(d_o.reshape(B * S, -1), dt)
    o, lse = torch.empty_like(g), torch.empty(B, nl, S, device="cuda")
    st = torch.cuda.current_stream()
    pkg.tp_layer_attn_fwd(dt, B, S, nl, dh, causal, x, o, lse, stream=st)
    runs = []
    for _ in range(2):
        dx, dsum = torch.full_like(x, 9.0), torch.full((B, nl, S), float("nan"), device="cuda")
        pkg.tp_layer_attn_bwd(dt, B, S, nl, dh, causal, x, o, lse, g, dx, dsum, stream=st)
        torch.cuda.synchronize()
        runs.append(dx)
    got = runs[0].cpu().numpy().reshape(B * S, 3, nl * dh)
    for i, nm in enumerate(("dQ", "dK", "dV")):
        assert oracle.max_rel_err(got[:, i], ref[:, i]) <= 1e-4, nm
    assert torch.equal(*runs)
