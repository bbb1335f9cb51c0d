"""GEMM groups on 128 x 256 tiles: forward passes that take them by themselves, with the first tokens above the line, column sums of weight gradients that are
cut over K, and independent GEMMs of one call at edges; against the oracle at the bf16 layer bound, layers twice over bit-identical."""
import numpy as np
import pytest

import oracle
import synthetic
import test_gpu_gemm_pairs as pairs
from synthetic.configs import small_variant
from test_few_token_plans import _groups

from gpu_util import compare, gpu_outputs, oracle_outputs, shard_inputs

pytestmark = pytest.mark.gpu


def _layer(cfg):
    d, sh = shard_inputs(cfg)
    a, b = gpu_outputs(cfg, d, sh, repeat=2)
    compare(cfg, a, oracle_outputs(cfg, d, sh))
    for k in a:
        assert np.array_equal(a[k], b[k]), k


def _on_wide_tiles(items, tune):
    import paper_2111_05972_amd as pkg
    need = {}
    for option in ("512", "256", "384", "128", "64", None):
        tune.set("gemm_group", option)
        need[option] = pkg.tp_layer_gemm_group_workspace_bytes(pkg.TPL_BF16, items)
    return need[None] == need["512"] and need["512"] not in [need[o] for o in ("256", "384", "128", "64")]


@pytest.mark.parametrize("hidden,seq", [(3712, 32), (3584, 64)])
def test_forward_that_takes_them(hidden, seq, tune):
    assert all(_on_wide_tiles(g, tune) for g in _groups(seq, hidden, hidden, 4 * hidden).values())
    print(f"\n[case] {seq} tokens of {hidden}", flush=True)
    _layer(small_variant(synthetic.CONFIGS[2], name="bf16-few-tokens", causal=True, row_epilogue=True, hidden=hidden, heads=hidden // 128, head_dim=128,
                         intermediate=4 * hidden, tp_degree=1, tp_rank=0, seq=seq, micro_batch=1))


@pytest.mark.parametrize("M,wide", [(104, True), (128, True), (136, False)])
def test_either_side_of_the_line(M, wide, tune):
    import torch
    import paper_2111_05972_amd as pkg
    print(f"\n[group] {M} rows of 12288 / 1536", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M)
    draw = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)   # noqa: E731
    for shapes in (((12288, 6144), (12288, 4608)), ((6144, 12288), (1536, 12288))):
        items = [(0, 0, M, N, K, draw(M, K), draw(K, N), torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)) for K, N in shapes]
        assert _on_wide_tiles(items, tune) == wide
        ws = torch.empty(pkg.tp_layer_gemm_group_workspace_bytes(pkg.TPL_BF16, items), dtype=torch.uint8, device="cuda")
        pkg.tp_layer_gemm_group(pkg.TPL_BF16, items, ws=ws, stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        for it in items:
            ref = it[5].double() @ it[6].double()
            assert ((it[7].double() - ref).abs().max() / ref.abs().max()).item() <= 2e-2


def test_column_sums_of_cut_tiles(tune):
    import paper_2111_05972_amd as pkg
    tune.set("gemm_group", "512")
    shape = dict(hidden=384, heads=6, head_dim=64, intermediate=1536, tp_degree=1, tp_rank=0, seq=500, micro_batch=22)
    M, H, I = 11000, 384, 1536
    weight_gradients = [(1, 0, I, H, M, None, None, None), (1, 0, H, H, M, None, None, None)]
    assert pkg.tp_layer_gemm_group_workspace_bytes(pkg.TPL_BF16, weight_gradients) >= 2 * 4 * H * H     # cut: float shares
    print(f"\n[case] {shape}", flush=True)
    _layer(small_variant(synthetic.CONFIGS[2], name="bf16-wide-tile-cut", causal=True, row_epilogue=True, **shape))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_data_and_weight_gradient(dtype, tune):
    pairs.test_data_and_weight_gradient(dtype, "512", tune)
