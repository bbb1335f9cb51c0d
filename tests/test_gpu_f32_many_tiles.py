"""Float layers whose launches have at least six 64-wide tiles to a compute unit (two stages in LDS instead of three), K of one step, of few and
of many, ragged in every dimension; against the oracle at the bound of the float layer tests, twice over bit-identical."""
import numpy as np
import pytest

import synthetic
from synthetic.configs import small_variant

from gpu_util import compare, gpu_outputs, oracle_outputs, shard_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    dict(hidden=264, heads=3, head_dim=88, intermediate=1060, tp_degree=1, tp_rank=0, seq=150, micro_batch=41),
    dict(hidden=32, heads=1, head_dim=32, intermediate=512, tp_degree=1, tp_rank=0, seq=251, micro_batch=70),
    dict(hidden=520, heads=4, head_dim=130, intermediate=2080, tp_degree=2, tp_rank=1, seq=111, micro_batch=61),
])
def test_layer(shape, tune):
    tune.set("gemm_group", "64")
    cfg = small_variant(synthetic.CONFIGS[1], name="f32-many-tiles", causal=True, row_epilogue=True, **shape)
    print(f"\n[case] {shape}", flush=True)
    d, sh = shard_inputs(cfg)
    a, b = gpu_outputs(cfg, d, sh, repeat=2)
    compare(cfg, a, oracle_outputs(cfg, d, sh))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
