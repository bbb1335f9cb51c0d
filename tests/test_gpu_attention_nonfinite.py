"""GPU: an infinity or a NaN in a later token does not reach earlier ones through the causal mask.  Float attention and bf16
attention at head sizes other than 64 and 128 leave masked positions out, also in the tile that the diagonal crosses, where a
matrix product would multiply a masked weight (zero) with the token's row.  Without a mask, an infinity in V gives infinities
and not NaN, also where a weight is multiplied in several terms.

The reference goes row by row over unmasked positions only, in float64; an element must be finite where the reference is, and
equal to it there at the parity tolerance (1e-4 and 2e-2 of the largest finite magnitude)."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu
S, NL = 200, 2


def _draw(seed, shape, dtype):
    return synthetic.quantize(synthetic.normal(seed, int(np.prod(shape)), 1.0), dtype).reshape(shape).astype(np.float32)


def _reference(qkv, d_o, dh, causal):
    """o, dqkv, lse of the S tokens, heads one by one."""
    w, scale = NL * dh, 1.0 / np.sqrt(dh)
    o, dqkv, lse = np.zeros((S, w)), np.zeros((S, 3 * w)), np.zeros((NL, S))
    for h in range(NL):
        Q, K, V = (qkv[:, i * w + h * dh:i * w + (h + 1) * dh].astype(np.float64) for i in range(3))
        dO, sl = d_o[:, h * dh:(h + 1) * dh].astype(np.float64), slice(h * dh, (h + 1) * dh)
        P, dS = np.zeros((S, S)), np.zeros((S, S))
        for i in range(S):
            n = i + 1 if causal else S
            s = K[:n] @ Q[i] * scale
            m = s.max()
            lse[h, i] = m + np.log(np.exp(s - m).sum())
            P[i, :n] = np.exp(s - lse[h, i])
            o[i, sl] = sum(P[i, j] * V[j] for j in range(n))
            dS[i, :n] = P[i, :n] * (V[:n] @ dO[i] - dO[i] @ o[i, sl])
            dqkv[i, sl] = sum(dS[i, j] * K[j] for j in range(n)) * scale
        for j in range(S):
            first = j if causal else 0
            dqkv[j, w + h * dh:w + (h + 1) * dh] = sum(dS[i, j] * Q[i] for i in range(first, S)) * scale
            dqkv[j, 2 * w + h * dh:2 * w + (h + 1) * dh] = sum(P[i, j] * dO[i] for i in range(first, S))
    return o, dqkv, lse


@pytest.mark.filterwarnings("ignore::RuntimeWarning")
@pytest.mark.parametrize("what,causal", [("q", True), ("k", True), ("v", True), ("do", True), ("v", False), ("do", False)])
@pytest.mark.parametrize("dtype,dh,chunk", [("f32", 36, None), ("f32", 64, None), ("f32", 128, None), ("bf16", 8, None), ("bf16", 40, "1"),
                                            ("bf16", 80, None), ("bf16", 96, "1"), ("bf16", 120, None)])
def test_masked_tokens_stay_out(dtype, dh, chunk, what, causal, tune):
    import torch
    import paper_2111_05972_amd as pkg
    tune.set("attn_chunk", chunk)
    dt, tol = (pkg.TPL_F32, 1e-4) if dtype == "f32" else (pkg.TPL_BF16, 2e-2)
    st = torch.cuda.current_stream()
    for token, value in ((150, np.inf), (45, np.nan), (95, -np.inf)):
        print(f"\n[attn] {dtype} dh={dh} chunk={chunk} causal={causal}: {value} in {what} of token {token}", flush=True)
        qkv, d_o = _draw(41, (S, 3 * NL * dh), dtype), _draw(42, (S, NL * dh), dtype)
        if what == "do":
            d_o[token, 3] = value
        else:
            qkv[token, "qkv".index(what) * NL * dh + 3] = value       # head 0; head 1 stays finite throughout
        o_ref, dqkv_ref, lse_ref = _reference(qkv, d_o, dh, causal)
        dev = lambda x: torch.from_numpy(x).to("cuda", torch.float32 if dtype == "f32" else torch.bfloat16)   # noqa: E731
        qkv_d, d_o_d = dev(qkv), dev(d_o)
        o, dqkv = torch.empty_like(d_o_d), torch.empty_like(qkv_d)
        lse, dsum = torch.empty(1, NL, S, device="cuda"), torch.empty(1, NL, S, device="cuda")
        ws = [torch.empty(max(pkg.tp_layer_attn_workspace_bytes(dt, 1, S, NL, dh, causal, bwd), 16), dtype=torch.uint8, device="cuda")
              if chunk else None for bwd in (False, True)]
        pkg.tp_layer_attn_fwd(dt, 1, S, NL, dh, causal, qkv_d, o, lse, ws=ws[0], stream=st)
        pkg.tp_layer_attn_bwd(dt, 1, S, NL, dh, causal, qkv_d, o, lse, d_o_d, dqkv, dsum, ws=ws[1], stream=st)
        torch.cuda.synchronize()
        for name, got, ref in (("o", o, o_ref), ("dqkv", dqkv, dqkv_ref), ("lse", lse[0], lse_ref)):
            got, fin = got.float().cpu().numpy(), np.isfinite(ref)
            assert np.isfinite(got[fin]).all(), (name, int((~np.isfinite(got[fin])).sum()))
            assert not np.isfinite(got[~fin]).any(), name
            if name == "o" and what == "v":
                assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]), name
            assert np.abs(got[fin] - ref[fin]).max() <= tol * max(1.0, np.abs(ref[fin]).max()), name
