"""Attention launches of many workgroups (head sizes 64 and 128), whose wavefronts own their rows: edges of a wavefront's 32 rows,
of a tile and of a block, one token, strips cut into chunks; forward and backward against the oracle's definitions, at the bound
of the other attention tests, and an infinity that the mask hides from every token up to 32 rows before it."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu

CASES = [(25, 1, 32, 64, None), (40, 33, 16, 64, None), (24, 130, 16, 64, None), (10, 193, 32, 128, None), (4, 300, 16, 64, "1"),
         (4, 300, 16, 128, "1")]


def _draw(seed, shape):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), 1.0), "bf16").reshape(shape)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_many_workgroups(case, causal, tune):
    import torch
    import paper_2111_05972_amd as pkg
    B, S, nl, dh, chunk = CASES[case]
    tune.set("attn_chunk", chunk)
    print(f"\n[attn] causal={causal} {CASES[case]}", flush=True)
    dt = pkg.TPL_BF16
    nbytes = max(pkg.tp_layer_attn_workspace_bytes(dt, B, S, nl, dh, causal, bwd) for bwd in (False, True))
    assert (nbytes > 0) == (chunk is not None)
    ws = torch.full((max(nbytes, 16) // 4,), float("nan"), dtype=torch.float32, device="cuda")
    qkv, d_o = _draw(30 + case, (B * S, 3 * nl * dh)), _draw(60 + case, (B * S, nl * dh))
    t = qkv.reshape(B, S, 3, nl, dh).astype(np.float64)
    Q, K, V = (t[:, :, i].transpose(0, 2, 1, 3) for i in range(3))
    O, P, LSE = oracle.attention_fwd(Q, K, V, causal)
    dQ, dK, dV = oracle.attention_bwd(Q, K, V, P, d_o.reshape(B, S, nl, dh).transpose(0, 2, 1, 3).astype(np.float64))
    ref = np.stack([a.transpose(0, 2, 1, 3) for a in (dQ, dK, dV)], axis=2).reshape(B * S, 3 * nl * dh)
    x, g = pkg.to_device(qkv, dt), pkg.to_device(d_o, dt)
    st = torch.cuda.current_stream()

    def run(x):
        o, dx = torch.full_like(g, 9.0), torch.full_like(x, 9.0)
        lse, dsum = (torch.empty(B, nl, S, dtype=torch.float32, device="cuda") for _ in range(2))
        pkg.tp_layer_attn_fwd(dt, B, S, nl, dh, causal, x, o, lse, ws=ws, stream=st)
        pkg.tp_layer_attn_bwd(dt, B, S, nl, dh, causal, x, o, lse, g, dx, dsum, ws=ws, stream=st)
        torch.cuda.synchronize()
        return o, lse, dx
    o, lse, dx = run(x)
    assert oracle.max_rel_err(o.float().cpu().numpy(), O.transpose(0, 2, 1, 3).reshape(B * S, nl * dh)) <= 2e-2
    assert np.abs(lse.cpu().numpy() - LSE).max() <= 2e-2
    got = dx.float().cpu().numpy()
    for i, nm in enumerate(("dQ", "dK", "dV")):
        sl = slice(i * nl * dh, (i + 1) * nl * dh)
        assert oracle.max_rel_err(got[:, sl], ref[:, sl]) <= 2e-2, nm
    again = run(x)
    assert torch.equal(o, again[0]) and torch.equal(lse, again[1]) and torch.equal(dx, again[2])
    if causal and S > 96:
        j = 32 * ((S - 1) // 32)                       # the first row of the last 32: rows before it are other wavefronts'
        y = x.view(B, S, 3, nl, dh).clone()
        y[0, j, 2, 0, 3] = float("inf")
        hit = run(y.view(B * S, 3 * nl * dh))[0]
        assert torch.equal(hit.view(B, S, nl * dh)[0, :j], o.view(B, S, nl * dh)[0, :j])


# forward without a mask: rows shared by two wavefronts where a workgroup per compute unit (256) has strips of more than 12 steps of 64
# keys (head size 64; 5 at 128), own rows where the strips are shorter, cut, or two workgroups share a unit
@pytest.mark.parametrize("B,S,nl,dh,chunk", [(1, 768, 3, 64, None), (1, 769, 3, 64, None), (2, 830, 18, 64, None), (1, 830, 37, 64, None), (1, 1000, 2, 64, "8"),
                                             (1, 320, 3, 128, None), (1, 321, 3, 128, None), (2, 449, 32, 128, None), (5, 449, 13, 128, None), (1, 700, 2, 128, "5")])
def test_forward_without_a_mask(B, S, nl, dh, chunk, tune):
    import torch
    import paper_2111_05972_amd as pkg
    tune.set("attn_chunk", chunk)
    print(f"\n[attn] {B} {S} {nl} {dh} chunk={chunk}", flush=True)
    dt = pkg.TPL_BF16
    nbytes = pkg.tp_layer_attn_workspace_bytes(dt, B, S, nl, dh, False, False) if chunk else 0
    ws = torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda") if chunk else None
    qkv = _draw(91, (B * S, 3 * nl * dh))
    Q, K, V = (qkv.reshape(B, S, 3, nl, dh).astype(np.float64)[:, :, i].transpose(0, 2, 1, 3) for i in range(3))
    O, _, LSE = oracle.attention_fwd(Q, K, V, False)
    x, runs = pkg.to_device(qkv, dt), []
    for _ in range(2):
        o, lse = torch.full((B * S, nl * dh), 9.0, dtype=x.dtype, device="cuda"), torch.empty(B, nl, S, dtype=torch.float32, device="cuda")
        pkg.tp_layer_attn_fwd(dt, B, S, nl, dh, False, x, o, lse, ws=ws, stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        runs.append((o, lse))
    assert oracle.max_rel_err(runs[0][0].float().cpu().numpy(), O.transpose(0, 2, 1, 3).reshape(B * S, nl * dh)) <= 2e-2
    assert np.abs(runs[0][1].cpu().numpy() - LSE).max() <= 2e-2
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])
