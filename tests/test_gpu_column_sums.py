"""Column sums in one launch (up to 1024 rows and 8 MB) and in two stages: row counts around the 128 row lanes and the line, column counts around the
32 columns of a workgroup.  A float sum of M terms is off by at most M 2^-24 of the sum of their magnitudes; the
stored bf16 adds 2^-8 of the result."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N", [(1, 8), (3, 32), (127, 40), (128, 64), (129, 24), (1023, 264), (1024, 2048), (1024, 4096), (1024, 4104), (1025, 264)])
def test_sums(M, N, dtype):
    import torch
    import paper_2111_05972_amd as pkg
    dt, td = (pkg.TPL_F32, torch.float32) if dtype == "f32" else (pkg.TPL_BF16, torch.bfloat16)
    print(f"\n[colsum] {dtype} {M} x {N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    x = (torch.randn(M, N, generator=g, device="cuda") + 0.5).to(td)
    ws = torch.empty(pkg.tp_layer_slice_epilogue_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    got = []
    for _ in range(2):
        out = torch.full((N + 16,), float("nan"), dtype=td, device="cuda")
        pkg.tp_layer_slice_epilogue_bwd(dt, pkg.TPL_ACT_NONE, M, N, x, None, None, out[8:N + 8], ws, stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert torch.isnan(out[:8]).all() and torch.isnan(out[N + 8:]).all()
        got.append(out[8:N + 8].double())
    assert torch.equal(got[0], got[1])
    ref = x.double().sum(0)
    bound = M * 2.0 ** -24 * x.double().abs().sum(0) + (2.0 ** -8 * ref.abs() if dtype == "bf16" else 0.0)
    assert ((got[0] - ref).abs() <= bound).all()
