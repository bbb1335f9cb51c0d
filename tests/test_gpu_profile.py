"""GPU: tp_layer_profile times the launches that a pass makes without it: the results are the same bits, and a layer whose
GEMMs go out as groups has one record per group."""
import pytest

import synthetic
from synthetic.configs import small_variant

pytestmark = pytest.mark.gpu

SHAPE = dict(hidden=512, heads=8, head_dim=64, intermediate=2048, tp_degree=2, tp_rank=1, seq=333, micro_batch=2, causal=True,
             row_epilogue=True)


@pytest.fixture
def group():
    import paper_2111_05972_amd as pkg
    yield lambda v: pkg.tp_layer_set_option("gemm_group", v)
    pkg.tp_layer_profile(0)
    pkg.tp_layer_set_option("gemm_group", None)


@pytest.mark.parametrize("option,launches", [(None, 4), ("0", 12)])
@pytest.mark.parametrize("dtype,side", [("bf16", False), ("bf16", True), ("f32", False)])
def test_profiled_pass_is_the_same_pass(dtype, side, option, launches, group):
    import torch
    import paper_2111_05972_amd as pkg
    group(option)
    cfg = small_variant(synthetic.CONFIGS[2], name="profile", **SHAPE)
    print(f"\n[profile] {dtype} side={side} gemm_group={option}", flush=True)
    dt, tdt = (pkg.TPL_BF16, torch.bfloat16) if dtype == "bf16" else (pkg.TPL_F32, torch.float32)
    layer = pkg.TpLayer(cfg.hidden, cfg.heads, cfg.tp_degree, cfg.tp_rank, cfg.seq, cfg.micro_batch, dt, cfg.causal,
                        cfg.row_epilogue, cfg.head_dim, cfg.intermediate, side_stream=side)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    rnd = lambda s, sigma=1.0: (torch.randn(*s, generator=g, device="cuda") * sigma).to(tdt)   # noqa: E731
    p = {k: rnd(s, 0.02) for k, s in layer.param_shapes().items()}
    x = [rnd((layer.M, layer.H)) for _ in range(4)]

    def step():
        y = layer.forward(p, x[0], x[1])
        grads, dx_a, dx_m = layer.backward(p, x[0], x[1], x[2], x[3])
        torch.cuda.synchronize()
        return {k: v.clone() for k, v in {"y_a": y[0], "y_m": y[1], "dx_a": dx_a, "dx_m": dx_m, **grads}.items()}
    plain = step()
    pkg.tp_layer_profile(1)
    timed = step()
    ms = pkg.tp_layer_profile_read()
    pkg.tp_layer_profile(0)
    assert len(ms) == launches and all(t > 0 for t in ms), ms
    for k in plain:
        assert torch.equal(plain[k], timed[k]), k
