"""D = rowsum(dO * O) where rows of dK are worked out again because a row beside them is not finite: it is a sum of eight partial sums, as in the
tiles, and no serial chain over the row.  Head sizes that keep weights in float, short strips, whose workgroups sum D themselves.

K is zero but for one infinity in token 1, so that scores are zero (P = 1 at a log-sum-exp of zero) and token 1's dK is not finite.  Query i has
a one in column i alone: dK[0][i] = (dP - D) of query i over sqrt(dh).  The terms of D are 1 and dh - 1 times 2^-25, each of which is lost
when it is added to the 1: a serial chain loses all of them.  dP = 1 + (dh - 1) 2^-25 rounded to float, from three elements of V.  A chunk of
eight terms loses at most its own seven, and a result on the order of 1 is rounded by 2^-24 in each of the at most five sums that
follow and in dP: |dP - D| <= 7 2^-25 + 6 2^-24."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,dh", [(24, 24), (40, 40), (65, 80), (104, 104), (120, 120)])
def test_finite_rows_beside_an_infinity(S, dh):
    import torch
    import paper_2111_05972_amd as pkg
    print(f"\n[attn] S={S} dh={dh}", flush=True)
    n = min(S, dh)
    z = lambda *shape: torch.zeros(*shape, dtype=torch.float64)   # noqa: E731
    q, k, v, o, d_o = (z(S, dh) for _ in range(5))
    q[range(n), range(n)] = 1.0
    k[1, dh - 1] = float("inf")
    d_o[:] = 2.0 ** -5
    o[:] = 2.0 ** -20
    d_o[:, 0], o[:, 0] = 1.0, 1.0
    terms = (d_o * o).sum(1)
    assert torch.equal(terms, torch.full((S,), 1.0 + (dh - 1) * 2.0 ** -25, dtype=torch.float64))
    rest = (terms[0].float().double() - 1.0).item()
    v[0, 0] = 1.0
    for column in (1, 2):                                   # what is left, times 2^5, in two bf16 pieces
        piece = torch.tensor(rest * 2.0 ** 5).to(torch.bfloat16).double().item()
        v[0, column], rest = piece, rest - piece * 2.0 ** -5
    assert rest == 0.0
    dev = lambda x: x.to(torch.bfloat16).cuda()   # noqa: E731
    qkv, o, d_o = dev(torch.cat([q, k, v], 1)), dev(o), dev(d_o)
    lse, dsum = torch.zeros(1, 1, S, device="cuda"), torch.empty(1, 1, S, device="cuda")
    dqkv = torch.full_like(qkv, float("nan"))
    pkg.tp_layer_attn_bwd(pkg.TPL_BF16, 1, S, 1, dh, True, qkv, o, lse, d_o, dqkv, dsum, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    dk = dqkv[:, dh:2 * dh].double().cpu() * dh ** 0.5
    assert not torch.isfinite(dk[1]).all()                  # the rows were worked out again
    assert torch.isfinite(dk[0]).all()
    assert dk[0, :n].abs().max().item() <= (7 * 2.0 ** -25 + 6 * 2.0 ** -24) * (1 + 2.0 ** -8)
