"""Which bf16 attention calls the matrix-core kernels take at the limit of their 32-bit offsets: a (batch, head) slice below
2 GiB at head sizes 64 and 128, and below 2 GiB with one tile of rows more at the others, whose columns past the head size
are marked by an offset of 2 GiB; and fewer than 2^32 threads in a launch.  Only those kernels cut strips, so with chunks
forced the workspace query tells (no GPU)."""
import pytest

BF16, TWO_GIB, TILE = 1, 1 << 31, 64


@pytest.mark.parametrize("dh,extra", [(64, 0), (128, 0), (32, TILE), (96, TILE), (120, TILE), (80, TILE)])
@pytest.mark.parametrize("nl", [1, 3])
def test_slice_limit(dh, extra, nl, tune):
    import paper_2111_05972_amd as pkg
    assert pkg.TPL_BF16 == BF16
    tune.set("attn_chunk", "1000")
    row = 3 * nl * dh * 2
    last = (TWO_GIB - 1) // row - extra                  # the longest sequence that is taken
    for bwd in (False, True):
        assert pkg.tp_layer_attn_workspace_bytes(BF16, 1, last, nl, dh, True, bwd) > 0
        assert pkg.tp_layer_attn_workspace_bytes(BF16, 1, last + 1, nl, dh, True, bwd) == 0


def test_launch_limit(tune):
    import paper_2111_05972_amd as pkg
    tune.set("attn_chunk", "8")
    # backward: 2 workgroups of 512 threads per 128 rows; 65535 heads x 64 blocks fit, 65 blocks do not
    for bwd in (False, True):
        assert pkg.tp_layer_attn_workspace_bytes(BF16, 65535, 64 * 128, 1, 8, True, bwd) > 0
        assert pkg.tp_layer_attn_workspace_bytes(BF16, 65535, 64 * 128 + 1, 1, 8, True, bwd) == 0
