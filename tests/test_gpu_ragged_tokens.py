"""GPU parity of the bf16 layer at token counts that are no multiple of 8: the tokens are the rows of the forward and
data-gradient GEMMs and the K of the weight gradients, so every tile kernel meets a ragged M and a ragged K."""
import pytest

import synthetic
from synthetic.configs import small_variant

from gpu_util import compare, gpu_outputs, oracle_outputs, shard_inputs

pytestmark = pytest.mark.gpu


def _run(name, seq, micro_batch):
    cfg = small_variant(synthetic.CONFIGS[2], name=name, hidden=512, heads=8, head_dim=64, intermediate=2064,
                        tp_degree=1, tp_rank=0, seq=seq, micro_batch=micro_batch, causal=True, row_epilogue=True)
    print(f"\n[case] {name} S={seq} B={micro_batch}", flush=True)
    d, sh = shard_inputs(cfg)
    compare(cfg, gpu_outputs(cfg, d, sh), oracle_outputs(cfg, d, sh))


# one token, fewer than a 16-byte chunk, one past a k-step, one short of and past a 128-row tile, several tiles
@pytest.mark.parametrize("seq,batch", [(1, 1), (7, 1), (33, 1), (127, 1), (129, 3), (1001, 1)])
def test_token_counts(seq, batch):
    _run("bf16-tokens", seq, batch)


# every tile kernel of the bf16 GEMM; K = 387 ends inside a k-step and inside a 64-k slot; with and without K shares
@pytest.mark.parametrize("shares", [None, "3"])
@pytest.mark.parametrize("tile", ["0", "1", "2", "3", "4", "5", "6", "7"])
def test_every_tile_kernel(tile, shares, tune):
    tune.set("gemm_tile", tile)
    tune.set("gemm_shares", shares)
    _run(f"bf16-tokens-tile{tile}", 129, 3)
