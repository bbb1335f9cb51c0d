"""Which tile the forward GEMM groups of few tokens go out on, told from the workspace they ask for (no GPU): 128 x 256 by turns where it leads, the tile
that is chosen otherwise where it was measured slower (8 tokens of 3136 / 3136 and of 11840 / 11840: small tiles, two rounds), and never above 128 rows."""
import pytest


def _groups(M, H, Hl, Il):
    gelu = 1
    up_qkv = [(0, 0, M, Il, H, None, None, None, None, gelu), (0, 0, M, 3 * Hl, H, None, None, None)]
    down_out = [(0, 0, M, H, Il, None, None, None), (0, 0, M, H, Hl, None, None, None)]
    return {"up_qkv": up_qkv, "down_out": down_out}


@pytest.mark.parametrize("M,H,T,group,tile", [
    (8, 3136, 1, "up_qkv", "128"), (8, 3136, 1, "down_out", "64"), (24, 3200, 1, "up_qkv", "128"), (8, 11840, 1, "up_qkv", "256"),
    (104, 12288, 8, "up_qkv", "512"), (104, 12288, 8, "down_out", "512"), (128, 12288, 8, "up_qkv", "512"), (128, 12288, 8, "down_out", "512"),
    (16, 10880, 2, "up_qkv", "512"), (64, 4608, 2, "up_qkv", "512"), (64, 4608, 2, "down_out", "512"),
    (136, 10880, 2, "up_qkv", "384"),
])
def test_tile(M, H, T, group, tile, tune):
    import paper_2111_05972_amd as pkg
    items = _groups(M, H, H // T, 4 * H // T)[group]
    need = {}
    for option in (None, "64", "128", "256", "384", "512"):
        tune.set("gemm_group", option)
        need[option] = pkg.tp_layer_gemm_group_workspace_bytes(pkg.TPL_BF16, items)
    assert need[None] == need[tile]
    assert (need[None] == need["512"]) == (tile == "512"), need
