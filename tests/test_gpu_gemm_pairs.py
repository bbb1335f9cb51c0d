"""Independent GEMMs of one call (tp_layer_gemm_group) against the oracle's definitions: a data gradient with GeLU' and the weight
gradient beside it, at edges of tiles and remainders, in one launch and, by option, one after another; and the layouts and
shapes that only single GEMMs take."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu


def _draw(seed, shape, sigma, dtype):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), sigma), dtype).reshape(shape)


@pytest.mark.parametrize("group", [None, "0", "256", "384"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_data_and_weight_gradient(dtype, group, tune):
    import torch
    import paper_2111_05972_amd as pkg
    tune.set("gemm_group", group)
    dt, tol = (pkg.TPL_BF16, 2e-2) if dtype == "bf16" else (pkg.TPL_F32, 1e-4)
    # tokens, input channels, output channels
    for si, (M, K, N) in enumerate([(8, 8, 8), (264, 136, 520), (1000, 1288, 264), (128, 64, 4104)]):
        print(f"\n[pair] {dtype} {group} {M} {K} {N}", flush=True)
        dy, w, x, u = (_draw(10 * si + q, s, sg, dtype) for q, (s, sg) in
                       enumerate([((M, N), 1.0), ((K, N), 0.05), ((M, K), 1.0), ((M, K), 1.0)]))
        d = {n: pkg.to_device(v, dt) for n, v in (("dy", dy), ("w", w), ("x", x), ("u", u))}
        dx, dw, tt = torch.empty_like(d["x"]), torch.empty_like(d["w"]), torch.empty(N, M, dtype=d["x"].dtype, device="cuda")
        items = [(0, 1, M, K, N, d["dy"], d["w"], dx, d["u"], pkg.TPL_EPI_DGELU), (1, 0, K, N, M, d["x"], d["dy"], dw)]
        # and both operands stored with K outermost: (x w)^T = w^T x^T, a layout that goes out by itself
        for it in (items, items + [(1, 1, N, M, K, d["w"], d["x"], tt)]):
            dx.zero_(), dw.zero_()
            ws = torch.empty(pkg.tp_layer_gemm_group_workspace_bytes(dt, it), dtype=torch.uint8, device="cuda")
            pkg.tp_layer_gemm_group(dt, it, ws=ws, stream=torch.cuda.current_stream())
            torch.cuda.synchronize()
            f = lambda t: t.float().cpu().numpy()   # noqa: E731
            dy64, w64, x64 = dy.astype(np.float64), w.astype(np.float64), x.astype(np.float64)
            assert oracle.max_rel_err(f(dx), (dy64 @ w64.T) * oracle.gelu_grad(u)) <= tol
            assert oracle.max_rel_err(f(dw), x64.T @ dy64) <= tol
        assert oracle.max_rel_err(f(tt), (x64 @ w64).T) <= tol
