"""GPU parity of the bf16 attention kernels at head sizes between their tile widths (32, 64, 96, 128): columns past the
head size must neither be read from the next head nor stored, with whole strips and with strips cut into chunks."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu


def _draw(seed, shape):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), 1.0), "bf16").reshape(shape)


@pytest.mark.parametrize("chunk", [None, "1"])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh", [8, 32, 40, 64, 72, 80, 96, 104, 128])
def test_head_sizes(dh, causal, chunk, tune):
    import torch
    import paper_2111_05972_amd as pkg
    tune.set("attn_chunk", chunk)
    dt, st, tol = pkg.TPL_BF16, torch.cuda.current_stream(), 2e-2
    for B, S, nl in [(1, 2, 1), (2, 65, 3), (1, 200, 2)]:
        print(f"\n[attn] dh={dh} causal={causal} chunk={chunk} B={B} S={S} nl={nl}", flush=True)
        qkv, d_o = _draw(21, (B * S, 3 * nl * dh)), _draw(22, (B * S, nl * dh))
        Q, K, V = (qkv.reshape(B, S, 3, nl, dh).astype(np.float64)[:, :, i].transpose(0, 2, 1, 3) for i in range(3))
        O, P, LSE = oracle.attention_fwd(Q, K, V, causal)
        rows = lambda x: x.transpose(0, 2, 1, 3).reshape(B * S, nl * dh)   # noqa: E731
        qkv_d = pkg.to_device(qkv, dt)
        o_d = torch.full((B * S, nl * dh), float("nan"), dtype=qkv_d.dtype, device="cuda")
        dqkv = torch.full_like(qkv_d, float("nan"))
        lse_d, dsum = torch.empty(B, nl, S, device="cuda"), torch.empty(B, nl, S, device="cuda")
        ws = [None, None]
        if chunk:
            ws = [torch.full((max(pkg.tp_layer_attn_workspace_bytes(dt, B, S, nl, dh, causal, bwd), 16) // 4,), float("nan"),
                             device="cuda") for bwd in (False, True)]
        pkg.tp_layer_attn_fwd(dt, B, S, nl, dh, causal, qkv_d, o_d, lse_d, ws=ws[0], stream=st)
        pkg.tp_layer_attn_bwd(dt, B, S, nl, dh, causal, qkv_d, o_d, lse_d, pkg.to_device(d_o, dt), dqkv, dsum, ws=ws[1], stream=st)
        torch.cuda.synchronize()
        assert oracle.max_rel_err(o_d.float().cpu().numpy(), rows(O)) <= tol
        assert np.abs(lse_d.cpu().numpy() - LSE).max() <= tol
        dO = d_o.reshape(B, S, nl, dh).transpose(0, 2, 1, 3).astype(np.float64)
        got, w = dqkv.float().cpu().numpy(), nl * dh
        for i, g in enumerate(oracle.attention_bwd(Q, K, V, P, dO)):
            assert oracle.max_rel_err(got[:, i * w:(i + 1) * w], rows(g)) <= tol, ("dQ", "dK", "dV")[i]
