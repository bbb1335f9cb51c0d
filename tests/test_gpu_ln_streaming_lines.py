"""LayerNorm stores y and dz with the non-temporal hint from 8 MB (bf16) and 2 MB (float) a tensor on, y in bf16 only of 2048 rows and more: which
kernel runs on either side of the lines, told from the last template parameter in its name (legible for float, and for bf16 rows of more than
1024), and its results against float64 at the parity bounds."""
import re

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,M,H,fwd,bwd", [
    ("bf16", 2048, 1952, False, False), ("bf16", 2048, 1960, True, True), ("bf16", 2047, 1960, False, True), ("bf16", 3875, 1032, False, False),
    ("bf16", 3876, 1032, True, True), ("bf16", 300, 16384, False, True), ("f32", 100, 512, False, False),
    ("f32", 488, 1024, False, False), ("f32", 489, 1024, True, True), ("f32", 61, 8192, False, False), ("f32", 62, 8192, True, True),
])
def test_hint(dtype, M, H, fwd, bwd):
    import torch
    from torch.profiler import ProfilerActivity, profile
    import paper_2111_05972_amd as pkg
    dt, td, tol = (pkg.TPL_F32, torch.float32, 1e-4) if dtype == "f32" else (pkg.TPL_BF16, torch.bfloat16, 2e-2)
    print(f"\n[ln] {dtype} {M} x {H}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + H)
    a, b, dy = (torch.randn(M, H, generator=g, device="cuda").to(td) for _ in range(3))
    gamma, beta = (torch.randn(H, generator=g, device="cuda").to(td) for _ in range(2))
    z, y, dz = (torch.full((M, H), float("nan"), dtype=td, device="cuda") for _ in range(3))
    mean, rstd = (torch.empty(M, device="cuda") for _ in range(2))
    dgamma, dbeta = torch.empty_like(gamma), torch.empty_like(beta)
    ws = torch.empty(pkg.tp_layer_ln_workspace_bytes(M, H), dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        pkg.tp_layer_ln_fwd(dt, M, H, a, b, gamma, beta, 1e-5, z, y, mean, rstd, stream=st)
        pkg.tp_layer_ln_bwd(dt, M, H, dy, z, mean, rstd, gamma, dz, dgamma, dbeta, ws, stream=st)
        torch.cuda.synchronize()
    names = [e.name for e in prof.events()]
    print(names, flush=True)
    hint = lambda part: [re.findall(r"Lb([01])E|(true|false)[,>]", n)[-1] in (("1", ""), ("", "true")) for n in names if part in n]   # noqa: E731
    assert hint("ln_fwd_") == [fwd] and hint("ln_bwd_") == [bwd], names
    zz, gm, d = z.double(), gamma.double(), dy.double()
    xh = (zz - zz.mean(1, keepdim=True)) / (zz.var(1, unbiased=False, keepdim=True) + 1e-5).sqrt()
    dx = d * gm
    ref = (dx - dx.mean(1, keepdim=True) - xh * (dx * xh).mean(1, keepdim=True)) / (zz.var(1, unbiased=False, keepdim=True) + 1e-5).sqrt()
    for got, want in ((y, xh * gm + beta.double()), (dz, ref), (dgamma, (d * xh).sum(0)), (dbeta, d.sum(0))):
        assert ((got.double() - want).abs().max() / want.abs().max()).item() <= tol


@pytest.mark.parametrize("M,H", [(7900, 512), (4000, 1024), (2500, 4104)])
def test_rows_are_the_same_on_both_sides(M, H):
    import torch
    import paper_2111_05972_amd as pkg
    td, st = torch.bfloat16, torch.cuda.current_stream()
    assert M * H * 2 >= 8_000_000 and M >= 2048
    print(f"\n[ln] bf16 {M} x {H}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(6)
    a, b, dy = (torch.randn(M, H, generator=g, device="cuda").to(td) for _ in range(3))
    gamma, beta = (torch.randn(H, generator=g, device="cuda").to(td) for _ in range(2))
    got = []
    for rows in (M, 1600):                          # with the hint on y, and without
        z, y, dz = (torch.full((rows, H), float("nan"), dtype=td, device="cuda") for _ in range(3))
        mean, rstd = (torch.empty(rows, device="cuda") for _ in range(2))
        dgamma, dbeta = torch.empty_like(gamma), torch.empty_like(beta)
        ws = torch.empty(pkg.tp_layer_ln_workspace_bytes(rows, H), dtype=torch.uint8, device="cuda")
        pkg.tp_layer_ln_fwd(pkg.TPL_BF16, rows, H, a[:rows], b[:rows], gamma, beta, 1e-5, z, y, mean, rstd, stream=st)
        pkg.tp_layer_ln_bwd(pkg.TPL_BF16, rows, H, dy[:rows], z, mean, rstd, gamma, dz, dgamma, dbeta, ws, stream=st)
        torch.cuda.synchronize()
        assert not torch.isnan(y).any() and not torch.isnan(dz).any()
        got.append((z, y, dz, mean, rstd))
    for whole, part in zip(*got):
        assert torch.equal(whole[:1600], part)
