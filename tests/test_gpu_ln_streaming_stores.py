"""LayerNorm of tensors above 100 MB, whose y and dz are stored without the non-temporal hint, against the same rows in a call below it: a row's
results do not depend on the other rows, so they are the same bits; rows of a wavefront (512, 1024 columns) and of a workgroup."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,M,H", [("f32", 3072, 8192), ("f32", 24480, 1024), ("bf16", 97792, 512), ("bf16", 12208, 4104)])
def test_rows_are_the_same_on_both_sides(dtype, M, H):
    import torch
    import paper_2111_05972_amd as pkg
    dt, td = (pkg.TPL_F32, torch.float32) if dtype == "f32" else (pkg.TPL_BF16, torch.bfloat16)
    size = 4 if dtype == "f32" else 2
    assert M * H * size > 100_000_000
    print(f"\n[ln] {dtype} {M} x {H}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    a, b, dy = (torch.randn(M, H, generator=g, device="cuda").to(td) for _ in range(3))
    gamma, beta = (torch.randn(H, generator=g, device="cuda").to(td) for _ in range(2))
    st = torch.cuda.current_stream()
    got = []
    for rows in (M, 1600):
        z, y, dz = (torch.full((rows, H), float("nan"), dtype=td, device="cuda") for _ in range(3))
        mean, rstd = (torch.empty(rows, device="cuda") for _ in range(2))
        dgamma, dbeta = torch.empty_like(gamma), torch.empty_like(beta)
        ws = torch.empty(pkg.tp_layer_ln_workspace_bytes(rows, H), dtype=torch.uint8, device="cuda")
        pkg.tp_layer_ln_fwd(dt, rows, H, a[:rows], b[:rows], gamma, beta, 1e-5, z, y, mean, rstd, stream=st)
        pkg.tp_layer_ln_bwd(dt, rows, H, dy[:rows], z, mean, rstd, gamma, dz, dgamma, dbeta, ws, stream=st)
        torch.cuda.synchronize()
        assert not torch.isnan(y).any() and not torch.isnan(dz).any()
        got.append((z, y, dz, mean, rstd))
    for whole, part in zip(*got):
        assert torch.equal(whole[:1600], part)
