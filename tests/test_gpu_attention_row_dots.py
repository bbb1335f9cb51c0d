"""D = rowsum(dO * O) of the attention backward on both sides of the line where it gets a kernel of its own: dQ, dK, dV against the oracle at
the bound of the other attention tests, D itself against float64 (products of bf16 pairs are exact in float, so a sum of dh of them is off by
at most dh 2^-24 of the sum of their magnitudes), run to run identical.  16 tile steps of 64 tokens are the line up to head size 64, 12
above: 1024 and 768 tokens are the last without the kernel, 1025 and 769 the first with it; ragged rows, head sizes that end inside a group of eight chunks."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu


def _draw(seed, shape):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), 1.0), "bf16").reshape(shape)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,S", [(8, 65), (24, 127), (32, 1024), (64, 1024), (64, 1025), (72, 63), (80, 768), (96, 769), (120, 129), (128, 768), (128, 769)])
def test_row_dots(dh, S, causal):
    import torch
    import paper_2111_05972_amd as pkg
    dt, st, B, nl = pkg.TPL_BF16, torch.cuda.current_stream(), 1, 2
    print(f"\n[attn] dh={dh} S={S} causal={causal}", flush=True)
    qkv, d_o = _draw(81, (B * S, 3 * nl * dh)), _draw(82, (B * S, nl * dh))
    Q, K, V = (qkv.reshape(B, S, 3, nl, dh).astype(np.float64)[:, :, i].transpose(0, 2, 1, 3) for i in range(3))
    O, P, LSE = oracle.attention_fwd(Q, K, V, causal)
    rows = lambda x: x.transpose(0, 2, 1, 3).reshape(B * S, nl * dh)   # noqa: E731
    x, g = pkg.to_device(qkv, dt), pkg.to_device(d_o, dt)
    o = pkg.to_device(rows(O).astype(np.float32), dt)
    lse = torch.from_numpy(np.ascontiguousarray(LSE.astype(np.float32))).cuda()
    got = []
    for _ in range(2):
        dqkv, dsum = torch.full_like(x, float("nan")), torch.full((B, nl, S), float("nan"), device="cuda")
        pkg.tp_layer_attn_bwd(dt, B, S, nl, dh, causal, x, o, lse, g, dqkv, dsum, stream=st)
        torch.cuda.synchronize()
        got.append((dqkv, dsum))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    terms = (o.float().cpu().numpy().astype(np.float64) * d_o).reshape(B, S, nl, dh).transpose(0, 2, 1, 3)
    assert (np.abs(got[0][1].cpu().numpy() - terms.sum(-1)) <= dh * 2.0 ** -24 * np.abs(terms).sum(-1)).all()
    ref = oracle.attention_bwd(Q, K, V, P, d_o.reshape(B, S, nl, dh).transpose(0, 2, 1, 3).astype(np.float64))
    w = nl * dh
    for i, r in enumerate(ref):
        assert oracle.max_rel_err(got[0][0].float().cpu().numpy()[:, i * w:(i + 1) * w], rows(r)) <= 2e-2, ("dQ", "dK", "dV")[i]
