"""The shard under HIP graph capture by the caller: tp_layer_fwd + tp_layer_bwd enqueue only kernels and (with
TPL_SIDE_STREAM, where the GEMMs are launched one by one) event records / waits, so a caller can capture a step into a graph
and replay it.  The replays must
reproduce the eager step bit for bit, also with eager work and synchronisations between them."""
import numpy as np
import pytest

import synthetic
from synthetic.configs import small_variant

from gpu_util import product_shard

pytestmark = pytest.mark.gpu

CASES = [
    ("bf16-one-stream", small_variant(synthetic.CONFIGS[2], name="graph-bf16", hidden=512, heads=8, intermediate=2048,
                                      tp_degree=2, tp_rank=1, seq=256, micro_batch=2, causal=True, row_epilogue=True), False, None),
    ("bf16-two-chains-grouped", small_variant(synthetic.CONFIGS[2], name="graph-bf16-side", hidden=512, heads=8, intermediate=2048,
                                      tp_degree=2, tp_rank=1, seq=256, micro_batch=2, causal=True, row_epilogue=True), True, None),
    ("f32-one-stream", small_variant(synthetic.CONFIGS[1], name="graph-f32", seq=64), False, None),
]
# launched one by one (option gemm_group 0), as layers with an operand of 2 GiB are: two chains fork from and join the captured stream
CASES += [("bf16-two-chains", CASES[1][1], True, "0"), ("f32-two-chains", CASES[2][1], True, "0"), ("f32-one-by-one", CASES[2][1], False, "0")]


@pytest.mark.parametrize("name,cfg,side,group", CASES, ids=[c[0] for c in CASES])
def test_step_captured_into_a_graph_replays_bit_identically(name, cfg, side, group, tune):
    import torch
    import paper_2111_05972_amd as pkg
    print(f"\n[graph] {name}", flush=True)
    tune.set("gemm_group", group)
    dt = pkg.TPL_F32 if cfg.dtype == "f32" else pkg.TPL_BF16
    d = synthetic.make_inputs(cfg)
    layer = pkg.TpLayer(cfg.hidden, cfg.heads, cfg.tp_degree, cfg.tp_rank, cfg.seq, cfg.micro_batch, dt, cfg.causal,
                        cfg.row_epilogue, cfg.head_dim, cfg.intermediate, side_stream=side)
    p = {k: pkg.to_device(v, dt) for k, v in product_shard(cfg, d).items()}
    x = {k: pkg.to_device(d[k], dt) for k in ("x_a", "x_m", "dy_a", "dy_m")}
    y_a, y_m = layer.empty_outputs()
    dx_a, dx_m = layer.empty_outputs()
    grads = layer.empty_grads()
    outs = {"y_a": y_a, "y_m": y_m, "dx_a": dx_a, "dx_m": dx_m, **grads}

    def step(st):
        layer.forward(p, x["x_a"], x["x_m"], y_a, y_m, stream=st)
        layer.backward(p, x["x_a"], x["x_m"], x["dy_a"], x["dy_m"], grads, dx_a, dx_m, stream=st)

    step(torch.cuda.current_stream())                       # eager: the expected values (and the one-off set-up calls)
    torch.cuda.synchronize()
    want = {k: v.clone() for k, v in outs.items()}
    cap = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    cap.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(cap):
        step(cap)                                           # warm-up on the capture stream
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=cap):
            step(torch.cuda.current_stream())
    torch.cuda.current_stream().wait_stream(cap)
    for rep in range(4):
        for v in outs.values():                             # eager work between the replays: wipe the outputs
            v.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for k, v in outs.items():
            if k in ("db_o", "db_dn") and not cfg.row_epilogue:
                continue
            assert torch.equal(v, want[k]), (name, rep, k)
        # an eager step between replays must not disturb the next one
        step(torch.cuda.current_stream())
        torch.cuda.synchronize()
