"""GPU parity of the float matrix-core kernels at the edges of their tiles: GEMM tiles of 32, 64 and 128 with remainders
of 4, and K cut into shares; attention at head sizes around multiples of 32 and sequence lengths around its 32-row tiles.

Tolerance: 2e-5 of the tensor's largest magnitude.  A float sum of K terms of one magnitude is off by about sqrt(K) 2^-24
of its own size (2.7e-6 at the K = 2052 used here), the softmax chain by a few of those; 1e-4 is what the layer promises."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu
TOL = 2e-5


def _draw(seed, shape, sigma=1.0):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), sigma), "f32").reshape(shape)


def _dev(x):
    import paper_2111_05972_amd as pkg
    return pkg.to_device(x, pkg.TPL_F32)


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(4, 4, 4), (36, 28, 132), (260, 132, 2052), (1028, 1156, 100), (2180, 2052, 68)])
def test_gemm_edges(M, N, K, ta, tb):
    import torch
    import paper_2111_05972_amd as pkg
    print(f"\n[gemm f32] ta={ta} tb={tb} M={M} N={N} K={K}", flush=True)
    A, B = _draw(1, (K, M) if ta else (M, K)), _draw(2, (N, K) if tb else (K, N))
    bias, resid, u = _draw(3, (N,)), _draw(4, (M, N)), _draw(5, (M, N))
    acc = (A.T if ta else A).astype(np.float64) @ (B.T if tb else B).astype(np.float64)
    ws = torch.empty(pkg.tp_layer_gemm_workspace_bytes(pkg.TPL_F32, M, N, K), dtype=torch.uint8, device="cuda")
    C, aux = torch.empty(M, N, device="cuda"), torch.empty(M, N, device="cuda")

    def gemm(**kw):
        C.fill_(float("nan"))
        pkg.tp_layer_gemm(pkg.TPL_F32, ta, tb, M, N, K, _dev(A), _dev(B), C, ws=ws, stream=torch.cuda.current_stream(), **kw)
        torch.cuda.synchronize()
        return C.cpu().numpy()
    assert oracle.max_rel_err(gemm(bias=_dev(bias), resid=_dev(resid)), acc + bias + resid) <= TOL
    assert oracle.max_rel_err(gemm(bias=_dev(bias), aux=aux, epi=pkg.TPL_EPI_GELU), oracle.gelu(acc + bias)) <= TOL
    assert oracle.max_rel_err(aux.cpu().numpy(), acc + bias) <= TOL
    assert oracle.max_rel_err(gemm(aux=_dev(u), epi=pkg.TPL_EPI_DGELU), acc * oracle.gelu_grad(u.astype(np.float64))) <= TOL


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh", [4, 32, 36, 64, 80, 96, 128])
def test_attention_edges(dh, causal):
    import torch
    import paper_2111_05972_amd as pkg
    dt, st = pkg.TPL_F32, torch.cuda.current_stream()
    for B, S, nl in [(1, 1, 1), (2, 31, 2), (1, 33, 3), (2, 130, 1), (1, 257, 2)]:
        print(f"\n[attn f32] causal={causal} B={B} S={S} nl={nl} dh={dh}", flush=True)
        qkv, d_o = _draw(11, (B * S, 3 * nl * dh)), _draw(12, (B * S, nl * dh))
        Q, K, V = (qkv.reshape(B, S, 3, nl, dh).astype(np.float64)[:, :, i].transpose(0, 2, 1, 3) for i in range(3))
        O, P, LSE = oracle.attention_fwd(Q, K, V, causal)
        rows = lambda x: x.transpose(0, 2, 1, 3).reshape(B * S, nl * dh)   # noqa: E731
        qkv_d, o_d = _dev(qkv), torch.empty(B * S, nl * dh, device="cuda")
        lse_d, dsum = torch.empty(B, nl, S, device="cuda"), torch.empty(B, nl, S, device="cuda")
        pkg.tp_layer_attn_fwd(dt, B, S, nl, dh, causal, qkv_d, o_d, lse_d, stream=st)
        dqkv = torch.full_like(qkv_d, float("nan"))
        pkg.tp_layer_attn_bwd(dt, B, S, nl, dh, causal, qkv_d, o_d, lse_d, _dev(d_o), dqkv, dsum, stream=st)
        torch.cuda.synchronize()
        assert oracle.max_rel_err(o_d.cpu().numpy(), rows(O)) <= TOL
        assert np.abs(lse_d.cpu().numpy() - LSE).max() <= TOL
        dO = d_o.reshape(B, S, nl, dh).transpose(0, 2, 1, 3).astype(np.float64)
        ref = np.concatenate([rows(g) for g in oracle.attention_bwd(Q, K, V, P, dO)], axis=1)
        if S > 1:       # at S = 1 dQ and dK are differences that cancel to zero
            assert oracle.max_rel_err(dqkv.cpu().numpy(), ref) <= TOL
