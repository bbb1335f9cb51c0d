"""Which launches of the bf16 attention backward work D = rowsum(dO * O) out in their workgroups and which get the row-dot kernel: at most 16, 6 and 4
workgroups to a compute unit up to head sizes 32, 64 and 128; above 64, strips of seven tiles and more, no last round that is up to a third full and,
without a mask, no third round.  On either side: the kernels that run, dQ, dK, dV against the oracle and D against float64, at the bounds of
test_gpu_attention_row_dots.py."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh,S,heads,causal,own", [
    (32, 64, 2048, True, True), (32, 64, 2049, False, False), (40, 33, 768, True, True), (40, 64, 769, True, False), (80, 64, 512, False, True),
    (128, 64, 513, False, False), (128, 128, 512, True, True), (104, 192, 257, False, False), (128, 448, 32, False, True), (128, 448, 40, True, False),
    (128, 448, 43, False, True), (120, 385, 40, False, False), (72, 384, 44, True, True), (128, 576, 56, False, False), (96, 520, 60, True, True),
])
def test_route(dh, S, heads, causal, own):
    import torch
    from torch.profiler import ProfilerActivity, profile
    import paper_2111_05972_amd as pkg
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines are stated for 256 compute units")
    print(f"\n[attn] dh={dh} S={S} heads={heads} causal={causal} own={own}", flush=True)
    dt, st = pkg.TPL_BF16, torch.cuda.current_stream()
    draw = lambda seed, *shape: synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), 1.0), "bf16").reshape(shape)   # noqa: E731
    w = heads * dh
    qkv, d_o = draw(91, S, 3 * w), draw(92, S, w)
    Q, K, V = (qkv.reshape(1, S, 3, heads, dh).astype(np.float64)[:, :, i].transpose(0, 2, 1, 3) for i in range(3))
    O, P, LSE = oracle.attention_fwd(Q, K, V, causal)
    rows = lambda x: x.transpose(0, 2, 1, 3).reshape(S, w)   # noqa: E731
    x, g, o = pkg.to_device(qkv, dt), pkg.to_device(d_o, dt), pkg.to_device(rows(O).astype(np.float32), dt)
    lse = torch.from_numpy(np.ascontiguousarray(LSE.astype(np.float32))).cuda()
    dqkv, dsum = torch.full_like(x, float("nan")), torch.full((1, heads, S), float("nan"), device="cuda")
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        pkg.tp_layer_attn_bwd(dt, 1, S, heads, dh, causal, x, o, lse, g, dqkv, dsum, stream=st)
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "attn" in e.name]
    assert len(names) == (1 if own else 2) and any("attn_dsum" in n for n in names) == (not own), names
    terms = (o.float().cpu().numpy().astype(np.float64) * d_o).reshape(1, S, heads, dh).transpose(0, 2, 1, 3)
    assert (np.abs(dsum.cpu().numpy() - terms.sum(-1)) <= dh * 2.0 ** -24 * np.abs(terms).sum(-1)).all()
    for i, r in enumerate(oracle.attention_bwd(Q, K, V, P, d_o.reshape(1, S, heads, dh).transpose(0, 2, 1, 3).astype(np.float64))):
        assert oracle.max_rel_err(dqkv[:, i * w:(i + 1) * w].float().cpu().numpy(), rows(r)) <= 2e-2, ("dQ", "dK", "dV")[i]
