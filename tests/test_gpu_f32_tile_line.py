"""Float GEMM groups on 64-wide tiles: two LDS stages from six workgroups to a compute unit on, three below it.  Which kernel runs on either side
of the line, told from its name, and its results against float64 at the parity bound; whole and ragged tiles, all layouts."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles,stages", [((768, 767), 3), ((768, 768), 2), ((700, 700), 3), ((1535, 1), 2), ((1504, 2), 3), ((1664, 2), 2)])
@pytest.mark.parametrize("ragged", [0, 24])
def test_stages(tiles, stages, ragged, tune):
    import torch
    from torch.profiler import ProfilerActivity, profile
    import paper_2111_05972_amd as pkg
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the line is stated for 256 compute units")
    tune.set("gemm_group", "64")
    print(f"\n[f32] {tiles} {ragged}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(sum(tiles) + ragged)
    items, want = [], []
    for i, t in enumerate(tiles):
        cols = next(c for c in (16, 8, 4, 3, 2, 1) if t % c == 0)
        M, N, K = 64 * (t // cols) - ragged, 64 * cols - ragged, 72
        ta, tb = ((1, 0), (0, 1))[i] if ragged else ((0, 0), (0, 1))[i]
        a = torch.randn(K, M, generator=g, device="cuda") if ta else torch.randn(M, K, generator=g, device="cuda")
        b = torch.randn(N, K, generator=g, device="cuda") if tb else torch.randn(K, N, generator=g, device="cuda")
        items.append((ta, tb, M, N, K, a, b, torch.full((M, N), float("nan"), device="cuda")))
        want.append((a.double().t() if ta else a.double()) @ (b.double().t() if tb else b.double()))
    ws = torch.empty(max(pkg.tp_layer_gemm_group_workspace_bytes(pkg.TPL_F32, items), 16), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        pkg.tp_layer_gemm_group(pkg.TPL_F32, items, ws=ws, stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "F32Tile" in e.name]
    assert len(names) == 1 and f"F32Tile<2, 2, 1, 1, 1, {stages}>" in names[0], names
    for it, w in zip(items, want):
        assert ((it[7].double() - w).abs().max() / w.abs().max()).item() <= 1e-4
