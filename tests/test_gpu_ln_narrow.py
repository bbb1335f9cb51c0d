"""GPU parity of LayerNorm over narrow rows (one wavefront per row, H <= 1024 and 4096 rows and more): the edges of each width class and the first
width past them; row counts around the eight rows of a workgroup, the 256 workgroups and the rows kept in flight; outputs
beyond the last row stay as they were; twice over bit-identical.  Tolerances are those of the wide rows."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu

CASES = [(4103, 8), (4100, 504), (4096, 512), (4097, 520), (4099, 1016), (4096, 1024), (4095, 1024), (4096, 1032), (6145, 1000),
         (8193, 136), (10241, 64)]


def _draw(seed, shape, sigma, dtype, mean=0.0):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), sigma) + np.float32(mean), dtype).reshape(shape)


@pytest.mark.parametrize("M,H", CASES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_narrow_rows(dtype, M, H):
    import torch
    import paper_2111_05972_amd as pkg
    dt, tol, st = (pkg.TPL_BF16, 2e-2, torch.cuda.current_stream()) if dtype == "bf16" else (pkg.TPL_F32, 1e-4, torch.cuda.current_stream())
    print(f"\n[ln narrow] {dtype} M={M} H={H}", flush=True)
    a, b, dy = _draw(950, (M, H), 1.0, dtype, mean=0.5), _draw(951, (M, H), 1.0, dtype), _draw(952, (M, H), 1.0, dtype)
    gamma, beta = _draw(953, (H,), 0.2, dtype, mean=1.0), _draw(954, (H,), 0.2, dtype)
    a_d, b_d, dy_d, g_d, be_d = (pkg.to_device(v, dt) for v in (a, b, dy, gamma, beta))
    f32 = lambda *s: torch.full(s, 7.0, dtype=torch.float32, device="cuda")       # noqa: E731
    like = lambda: torch.full((M + 3, H), 7.0, dtype=a_d.dtype, device="cuda")    # noqa: E731
    runs = []
    for _ in range(2):
        z, y, dz, mean, rstd, dg, db = like(), like(), like(), f32(M + 3), f32(M + 3), torch.empty_like(g_d), torch.empty_like(g_d)
        ws = torch.empty(pkg.tp_layer_ln_workspace_bytes(M, H), dtype=torch.uint8, device="cuda")
        pkg.tp_layer_ln_fwd(dt, M, H, a_d, b_d, g_d, be_d, 1e-5, z, y, mean, rstd, stream=st)
        pkg.tp_layer_ln_bwd(dt, M, H, dy_d, z, mean, rstd, g_d, dz, dg, db, ws, stream=st)
        torch.cuda.synchronize()
        runs.append({"z": z, "y": y, "mean": mean, "rstd": rstd, "dz": dz, "dgamma": dg, "dbeta": db})
    y_ref, z_ref, mean_ref, rstd_ref = oracle.layernorm_fwd(a, b, gamma, beta, 1e-5)
    dz_ref, dg_ref, db_ref = oracle.layernorm_bwd(dy, z_ref, mean_ref, rstd_ref, gamma)
    ref = {"z": z_ref, "y": y_ref, "mean": mean_ref, "rstd": rstd_ref, "dz": dz_ref, "dgamma": dg_ref, "dbeta": db_ref}
    for k, v in runs[0].items():
        got = v.float().cpu().numpy()
        if k not in ("dgamma", "dbeta"):
            assert (got[M:] == 7.0).all(), k
            got = got[:M]
        err = oracle.max_rel_err(got, ref[k])
        assert err <= tol, (k, err)
        assert torch.equal(v, runs[1][k]), k
