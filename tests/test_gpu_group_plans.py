"""GPU parity of bf16 layers on either side of the lines of the group planner: up to 64 rows the small tiles are ranked with what their
columns read again (widths of the 4096 / 1024 shard), and groups with weight gradients leave the 256-wide tiles where their lead is
small.  Against the oracle, at the bound of every bf16 layer test, and twice over bit-identical."""
import numpy as np
import pytest

import synthetic
from synthetic.configs import small_variant

from gpu_util import compare, gpu_outputs, oracle_outputs, shard_inputs

pytestmark = pytest.mark.gpu

WIDE = dict(hidden=4096, heads=32, head_dim=128, intermediate=16384, tp_degree=4, tp_rank=1)
NARROW = dict(hidden=1024, heads=16, head_dim=64, intermediate=4096, tp_degree=1, tp_rank=0)


@pytest.mark.parametrize("widths,seq", [(WIDE, 33), (WIDE, 64), (WIDE, 65), (NARROW, 273), (NARROW, 1000)])
def test_layer_at_the_lines(widths, seq):
    cfg = small_variant(synthetic.CONFIGS[5], name=f"bf16-plans-{seq}", seq=seq, micro_batch=1, causal=True, row_epilogue=True, **widths)
    print(f"\n[case] {cfg.hidden} S={seq}", flush=True)
    d, sh = shard_inputs(cfg)
    a, b = gpu_outputs(cfg, d, sh, repeat=2)
    compare(cfg, a, oracle_outputs(cfg, d, sh))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
