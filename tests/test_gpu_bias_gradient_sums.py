"""GPU: the bias gradients that ride in a group's weight gradients lose no more to float rounding than the column-sum kernels
do, which add 64 rows at a time.  db_o and db_dn are column sums of the upstream gradients as given, so the exact values are
known.  The root mean square error over the columns may be 1.1 times that of the column-sum kernels (option gemm_group 0):
over 1024 columns such a figure is itself uncertain by 2 %.  bf16: the rows come as +a and, shuffled, -a, so that the exact
sum is zero and rounding the result to bf16 does not hide its error."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture
def group():
    import paper_2111_05972_amd as pkg
    yield lambda v: pkg.tp_layer_set_option("gemm_group", v)
    pkg.tp_layer_set_option("gemm_group", None)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rounding_of_the_sums(dtype, group):
    import torch
    import paper_2111_05972_amd as pkg
    H, S, B = (2048, 128, 256) if dtype == "bf16" else (1024, 128, 128)     # wide enough that the sums are not cut over K
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    M, g = S * B, torch.Generator(device="cuda")
    g.manual_seed(7)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dt)   # noqa: E731
    x, dys = rnd(M, H), []
    for _ in range(2):
        d = rnd(M, H)
        if dtype == "bf16":
            d[M // 2:] = -d[:M // 2][torch.randperm(M // 2, generator=g, device="cuda")]
        dys.append(d)

    def errors(tile):
        group(tile)
        layer = pkg.TpLayer(H, H // 64, 1, 0, S, B, pkg.TPL_BF16 if dtype == "bf16" else pkg.TPL_F32, False, True, 64, H)
        params = {k: torch.full(s, 0.01, dtype=dt, device="cuda") for k, s in layer.param_shapes().items()}
        layer.forward(params, x, x)
        grads, _, _ = layer.backward(params, x, x, *dys)
        torch.cuda.synchronize()
        return [(grads[k].double() - d.double().sum(0)).pow(2).mean().sqrt().item() for k, d in zip(("db_o", "db_dn"), dys)]
    alone, got = errors("0"), {}
    for tile in ("64", "128", "192"):
        got[tile] = errors(tile)
        print(f"\n[bias] {dtype} tile {tile}: rms error {got[tile]}, column-sum kernels {alone}", flush=True)
    for tile, e in got.items():
        assert all(a <= 1.1 * b for a, b in zip(e, alone)), (tile, e, alone)
