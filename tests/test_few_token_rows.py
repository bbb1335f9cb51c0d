"""Forward GEMM groups of few tokens do not go out on 128 x 256 tiles where the rows of their largest weight are not whole cache lines, or in fewer workgroups
than nine sixteenths of 256 compute units (4816: 133, 5312: 146), told from the workspace they ask for (no GPU).  The lines are the largest
weight's, not the other's: {up, qkv} of 6432 has rows of 25728 elements beside rows of 19296."""
import pytest

from test_few_token_plans import _groups


@pytest.mark.parametrize("M,H,T,group,tile", [
    (64, 8944, 1, "down_out", "256"), (56, 9664, 1, "down_out", "512"), (16, 4024, 1, "down_out", "256"), (48, 6432, 1, "down_out", "384"),
    (16, 5768, 1, "up_qkv", "384"), (48, 6432, 1, "up_qkv", "512"), (104, 12288, 8, "down_out", "512"),
    (80, 4816, 1, "up_qkv", "384"), (32, 10304, 2, "up_qkv", "384"), (32, 5312, 1, "up_qkv", "512"),
])
def test_whole_lines(M, H, T, group, tile, tune):
    import paper_2111_05972_amd as pkg
    items = _groups(M, H, H // T, 4 * H // T)[group]
    need = {}
    for option in (None, "256", "384", "512"):
        tune.set("gemm_group", option)
        need[option] = pkg.tp_layer_gemm_group_workspace_bytes(pkg.TPL_BF16, items)
    assert need[None] == need[tile]
    assert (need[None] == need["512"]) == (tile == "512"), need
