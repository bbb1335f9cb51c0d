"""dK and dV of launches of few workgroups, whose wavefronts pass the probabilities on through LDS one sub-tile of 32 queries late:
strips of 1 to 8 tiles of 64 queries (three LDS stages), a last sub-tile that is full, ragged or missing, strips cut into chunks
of one and of five tiles; against the oracle at the bound of the other attention tests, and run to run identical."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu


def _draw(seed, shape):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), 1.0), "bf16").reshape(shape)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,chunk", [(128, None), (128, "1"), (128, "5"), (64, None), (64, "5"), (80, None), (104, "1"), (32, None)])
def test_dk_dv(dh, chunk, causal, tune):
    import torch
    import paper_2111_05972_amd as pkg
    tune.set("attn_chunk", chunk)
    dt, st = pkg.TPL_BF16, torch.cuda.current_stream()
    # not two tokens: O rounded to bf16 moves D = sum dO O by up to 2^-9 sum |dO O| (0.1 at 64 columns), and there the exact dS can
    # be as small
    for B, S, nl in [(1, 31, 2), (2, 32, 1), (1, 33, 1), (1, 97, 2), (1, 160, 1), (1, 225, 1), (1, 320, 2), (1, 512, 1)]:
        print(f"\n[attn] dh={dh} causal={causal} chunk={chunk} B={B} S={S} nl={nl}", flush=True)
        qkv, d_o = _draw(71, (B * S, 3 * nl * dh)), _draw(72, (B * S, nl * dh))
        Q, K, V = (qkv.reshape(B, S, 3, nl, dh).astype(np.float64)[:, :, i].transpose(0, 2, 1, 3) for i in range(3))
        O, P, LSE = oracle.attention_fwd(Q, K, V, causal)
        rows = lambda x: x.transpose(0, 2, 1, 3).reshape(B * S, nl * dh)   # noqa: E731
        x, g = pkg.to_device(qkv, dt), pkg.to_device(d_o, dt)
        o = pkg.to_device(rows(O).astype(np.float32), dt)
        lse = torch.from_numpy(np.ascontiguousarray(LSE.astype(np.float32))).cuda()
        ws = None
        if chunk:
            ws = torch.full((max(pkg.tp_layer_attn_workspace_bytes(dt, B, S, nl, dh, causal, True), 16) // 4,), float("nan"), device="cuda")
        got = []
        for _ in range(2):
            dqkv, dsum = torch.full_like(x, float("nan")), torch.empty(B, nl, S, device="cuda")
            pkg.tp_layer_attn_bwd(dt, B, S, nl, dh, causal, x, o, lse, g, dqkv, dsum, ws=ws, stream=st)
            torch.cuda.synchronize()
            got.append(dqkv)
        assert torch.equal(got[0], got[1])
        ref = oracle.attention_bwd(Q, K, V, P, d_o.reshape(B, S, nl, dh).transpose(0, 2, 1, 3).astype(np.float64))
        w = nl * dh
        for i, r in enumerate(ref):
            assert oracle.max_rel_err(got[0].float().cpu().numpy()[:, i * w:(i + 1) * w], rows(r)) <= 2e-2, ("dQ", "dK", "dV")[i]
