"""Single bf16 GEMMs on the 256 x 256 tile whose wavefronts take turns at the matrix cores, against the oracle's definitions at the
bound of the other GEMM tests: forced (option gemm_tile 8) over edges of a tile in every dimension, K whole and in shares, every
epilogue; and by the library's own choice, at shapes with remainders where it takes this tile, with the workspace it asks for."""
import numpy as np
import pytest

import oracle
import synthetic
from test_gpu_kernels import _check_gemms

pytestmark = pytest.mark.gpu

SHAPES = [(8, 8, 8), (256, 256, 64), (264, 248, 72), (520, 264, 1096), (248, 776, 2056), (1000, 520, 136)]


@pytest.mark.parametrize("shares", [None, "2", "5"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("epi", ["none", "bias", "bias_resid", "gelu", "dgelu"])
def test_forced(shares, ta, tb, epi, tune):
    _check_gemms("bf16", "8", shares, ta, tb, epi, SHAPES, tune)


def _quantized(seed, shape, sigma):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), sigma), "bf16").reshape(shape)


# K shares of whole tiles where M or N is no multiple of 256 are no multiple of M x N sums: the workspace tells that the tile is taken
@pytest.mark.parametrize("ta,tb,M,N,K", [(0, 0, 2040, 2552, 4104), (0, 1, 2040, 2552, 4104), (1, 0, 2040, 2552, 4104), (0, 0, 2040, 15352, 1032),
                                         (0, 1, 3064, 4600, 3080), (1, 0, 2040, 4600, 3080)])
@pytest.mark.parametrize("epi", ["none", "bias_resid", "gelu_resid"])
def test_own_choice(ta, tb, M, N, K, epi, tune):
    import torch
    import paper_2111_05972_amd as pkg
    print(f"\n[gemm] ta={ta} tb={tb} {M} {N} {K} {epi}", flush=True)
    tune.set("gemm_tile", None)
    dt = pkg.TPL_BF16
    nbytes = pkg.tp_layer_gemm_workspace_bytes(dt, M, N, K)
    if K == 4104:
        tiles = -(-M // 256) * -(-N // 256)
        assert nbytes % (tiles * 65536 * 4) == 0 and nbytes % (M * N * 4) != 0
    A, Bm = _quantized(11, (K, M) if ta else (M, K), 1.0), _quantized(12, (N, K) if tb else (K, N), 0.02)
    ref = (A.T if ta else A).astype(np.float32) @ (Bm.T if tb else Bm).astype(np.float32)   # float sums of up to 4104 terms: 1e-5
    kw = {}
    if epi != "none":
        bias, resid = _quantized(13, (N,), 0.5), _quantized(14, (M, N), 1.0)
        kw.update(bias=pkg.to_device(bias, dt), resid=pkg.to_device(resid, dt))
        ref = ref + bias + resid
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    if epi == "gelu_resid":
        aux = torch.full_like(C, float("nan"))
        kw.update(aux=aux, epi=pkg.TPL_EPI_GELU)
    ws = torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda")
    a, b = pkg.to_device(A, dt), pkg.to_device(Bm, dt)
    runs = []
    for _ in range(2):
        pkg.tp_layer_gemm(dt, ta, tb, M, N, K, a, b, C, ws=ws, stream=torch.cuda.current_stream(), **kw)
        torch.cuda.synchronize()
        runs.append(C.clone())
    assert torch.equal(*runs)
    if epi == "gelu_resid":
        assert oracle.max_rel_err(aux.float().cpu().numpy(), ref) <= 2e-2
        ref = oracle.gelu(ref)
    assert oracle.max_rel_err(C.float().cpu().numpy(), ref) <= 2e-2
