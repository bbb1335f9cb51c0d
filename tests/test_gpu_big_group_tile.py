"""GPU parity of layers whose GEMM groups go out on 256 x 256 and 256 x 128 tiles (option gemm_group 256, 384): edges of a tile in every
dimension, token counts that are no multiple of the 64 k of a step (K of the weight gradients), K shares, and a list whose
last tiles alone are cut; bias gradients as column sums of whole and of cut tiles.  Against the oracle, at the bound of every
bf16 layer test, and twice over bit-identical."""
import numpy as np
import pytest

import synthetic
from synthetic.configs import small_variant

from gpu_util import compare, gpu_outputs, oracle_outputs, shard_inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    dict(hidden=64, heads=1, head_dim=64, intermediate=72, tp_degree=1, tp_rank=0, seq=1, micro_batch=1),
    dict(hidden=256, heads=4, head_dim=64, intermediate=512, tp_degree=2, tp_rank=1, seq=256, micro_batch=1),
    dict(hidden=264, heads=3, head_dim=88, intermediate=520, tp_degree=1, tp_rank=0, seq=257, micro_batch=1),
    dict(hidden=1040, heads=10, head_dim=104, intermediate=2096, tp_degree=2, tp_rank=0, seq=129, micro_batch=5),
    # dx of the MLP block: 86 tiles; dx of the attention block: 53 tiles whole and 33 in two K shares; dW in five
    dict(hidden=384, heads=6, head_dim=64, intermediate=1536, tp_degree=1, tp_rank=0, seq=500, micro_batch=22),
]


@pytest.mark.parametrize("epilogue", [True, False])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("tile", ["256", "384"])
def test_layer_on_big_tiles(tile, shape, epilogue, tune):
    tune.set("gemm_group", tile)
    cfg = small_variant(synthetic.CONFIGS[2], name=f"bf16-group-{tile}", causal=True, row_epilogue=epilogue, **SHAPES[shape])
    print(f"\n[case] {tile} {SHAPES[shape]} epi={epilogue}", flush=True)
    d, sh = shard_inputs(cfg)
    a, b = gpu_outputs(cfg, d, sh, repeat=2)
    compare(cfg, a, oracle_outputs(cfg, d, sh))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
