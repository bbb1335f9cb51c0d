"""GPU parity of the layer with its independent GEMMs in one launch per level (option gemm_group): every group tile, over
shapes with remainders in every dimension, with and without K shares, and the bias gradients that ride in the weight
gradients' launches; against the oracle, and twice over bit-identical."""
import numpy as np
import pytest

import synthetic
from synthetic.configs import small_variant

from gpu_util import compare, gpu_outputs, oracle_outputs, shard_inputs

pytestmark = pytest.mark.gpu
C = synthetic.CONFIGS

SHAPES = [
    # narrower than any tile; long K for the weight gradients (shares); one tile and a bit in every dimension
    dict(hidden=64, heads=1, head_dim=64, intermediate=72, tp_degree=1, tp_rank=0, seq=5, micro_batch=1),
    dict(hidden=128, heads=2, head_dim=64, intermediate=256, tp_degree=2, tp_rank=1, seq=999, micro_batch=3),
    dict(hidden=520, heads=5, head_dim=104, intermediate=1048, tp_degree=1, tp_rank=0, seq=131, micro_batch=2),
]


@pytest.fixture
def group():
    import paper_2111_05972_amd as pkg
    yield lambda v: pkg.tp_layer_set_option("gemm_group", v)
    pkg.tp_layer_set_option("gemm_group", None)


@pytest.mark.parametrize("epilogue", [True, False])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("tile", ["64", "128", "192", None])
def test_group_tiles(tile, shape, epilogue, group, tune):
    group(tile)
    cfg = small_variant(C[2], name=f"bf16-group-{tile}", causal=True, row_epilogue=epilogue, **SHAPES[shape])
    print(f"\n[case] {cfg.name} {SHAPES[shape]} epi={epilogue}", flush=True)
    d, sh = shard_inputs(cfg)
    a, b = gpu_outputs(cfg, d, sh, repeat=2)
    compare(cfg, a, oracle_outputs(cfg, d, sh))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
