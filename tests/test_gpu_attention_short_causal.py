"""Causal forward of short strips (1 to 3 tile steps on wavefronts that own their rows, longer ones on shared rows) against the oracle at the bound
of the other attention tests: both sides of 64, 128 and 192 tokens, a single token, every row written."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("S", [1, 33, 64, 65, 128, 129, 192, 193])
def test_forward(S, dh):
    import torch
    import paper_2111_05972_amd as pkg
    dt, B, nl = pkg.TPL_BF16, 2, 3
    print(f"\n[attn] dh={dh} S={S}", flush=True)
    qkv = synthetic.quantize(synthetic.normal(91, B * S * 3 * nl * dh, 1.0), "bf16").reshape(B * S, 3 * nl * dh)
    Q, K, V = (qkv.reshape(B, S, 3, nl, dh).astype(np.float64)[:, :, i].transpose(0, 2, 1, 3) for i in range(3))
    O, _, LSE = oracle.attention_fwd(Q, K, V, True)
    x = pkg.to_device(qkv, dt)
    o = torch.full((B * S, nl * dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, nl, S), float("nan"), device="cuda")
    pkg.tp_layer_attn_fwd(dt, B, S, nl, dh, True, x, o, lse, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert oracle.max_rel_err(o.float().cpu().numpy(), O.transpose(0, 2, 1, 3).reshape(B * S, nl * dh)) <= 2e-2
    assert oracle.max_rel_err(lse.cpu().numpy(), LSE) <= 1e-4
