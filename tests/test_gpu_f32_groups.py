"""GPU parity of the float layer with its independent GEMMs in one launch per level (option gemm_group; 192 stands for the
32-wide tile there): every tile, over shapes with remainders of 4 in every dimension, with and without K shares, and the
bias gradients that ride in the weight gradients' launches; against the oracle at the layer's float tolerance, and twice
over bit-identical."""
import numpy as np
import pytest

import synthetic
from synthetic.configs import small_variant

from gpu_util import compare, gpu_outputs, oracle_outputs, shard_inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    dict(hidden=20, heads=1, head_dim=20, intermediate=12, tp_degree=1, tp_rank=0, seq=5, micro_batch=1),       # inside one tile
    dict(hidden=136, heads=2, head_dim=68, intermediate=264, tp_degree=2, tp_rank=1, seq=681, micro_batch=3),   # long K: shares
    dict(hidden=260, heads=5, head_dim=52, intermediate=516, tp_degree=1, tp_rank=0, seq=131, micro_batch=2),
]


@pytest.fixture
def group():
    import paper_2111_05972_amd as pkg
    yield lambda v: pkg.tp_layer_set_option("gemm_group", v)
    pkg.tp_layer_set_option("gemm_group", None)


@pytest.mark.parametrize("epilogue", [True, False])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("tile", ["64", "128", "192", None])
def test_group_tiles(tile, shape, epilogue, group):
    group(tile)
    cfg = small_variant(synthetic.CONFIGS[1], name=f"f32-group-{tile}", causal=True, row_epilogue=epilogue, **SHAPES[shape])
    print(f"\n[case] {cfg.name} {SHAPES[shape]} epi={epilogue}", flush=True)
    d, sh = shard_inputs(cfg)
    a, b = gpu_outputs(cfg, d, sh, repeat=2)
    compare(cfg, a, oracle_outputs(cfg, d, sh))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
