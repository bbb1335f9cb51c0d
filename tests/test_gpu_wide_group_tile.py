"""GPU parity of layers whose GEMM groups go out on 128 x 256 tiles (option gemm_group 512): edges of a tile in every dimension, more rows than
one tile has, K shares, column sums of whole and of cut tiles; and of the forward passes that take it by themselves (at most 128 tokens of a
wide layer).  Against the oracle, at the bound of every bf16 layer test, and twice over bit-identical."""
import numpy as np
import pytest

import synthetic
from synthetic.configs import small_variant

from gpu_util import compare, gpu_outputs, oracle_outputs, shard_inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    dict(hidden=64, heads=1, head_dim=64, intermediate=72, tp_degree=1, tp_rank=0, seq=1, micro_batch=1),
    dict(hidden=256, heads=4, head_dim=64, intermediate=512, tp_degree=2, tp_rank=1, seq=128, micro_batch=1),
    dict(hidden=264, heads=3, head_dim=88, intermediate=520, tp_degree=1, tp_rank=0, seq=129, micro_batch=1),
    dict(hidden=1040, heads=10, head_dim=104, intermediate=2096, tp_degree=2, tp_rank=0, seq=127, micro_batch=5),
    dict(hidden=2048, heads=16, head_dim=128, intermediate=8192, tp_degree=1, tp_rank=0, seq=63, micro_batch=2),
]


@pytest.mark.parametrize("tile", ["512", None])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_layer_on_wide_tiles(tile, shape, tune):
    tune.set("gemm_group", tile)
    cfg = small_variant(synthetic.CONFIGS[2], name="bf16-wide-tile", causal=True, row_epilogue=True, **SHAPES[shape])
    print(f"\n[case] {tile} {SHAPES[shape]}", flush=True)
    d, sh = shard_inputs(cfg)
    a, b = gpu_outputs(cfg, d, sh, repeat=2)
    compare(cfg, a, oracle_outputs(cfg, d, sh))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
