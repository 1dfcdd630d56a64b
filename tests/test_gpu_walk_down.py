"""dK/dV of causal sequences long enough to be walked from their last row block down (head dims 192, 256 and 512), alone and beside a short
one in a call of several groups: against 64-bit arithmetic, and the two calls bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _exact(q, k, v, do, scale):
    """dK, dV of one KV head in float64; q, do (n, G, d), k, v (n, d)"""
    import torch
    n, G, d = q.shape
    hidden = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
    dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    for g in range(G):
        p = ((q[:, g] @ k.t()) * scale).masked_fill_(hidden, float("-inf")).softmax(1)
        dv += p.t() @ do[:, g]
        ds = do[:, g] @ v.t()
        ds = p * (ds - (p * ds).sum(1, keepdim=True)) * scale
        dk += ds.t() @ q[:, g]
    return dk, dv


# 4 M elements of Q rows of a KV head is where the direction changes: just below, there, and past it with partial tiles and blocks
@pytest.mark.parametrize("d,H,Hk,P", [(192, 8, 1, 2730), (192, 8, 1, 2735), (256, 8, 1, 2047), (256, 16, 2, 2049), (512, 8, 1, 1023),
                                      (512, 16, 2, 1031), (512, 8, 1, 1024)])
def test_long_causal_rows(d, H, Hk, P):
    import torch
    from paper_2605_15422_amd import binding as B
    print("case walk down", d, H, Hk, P, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(d + P)
    small = 150
    q, k, v, do = (torch.randn((P + small, h, d), generator=gen, device="cuda").bfloat16() for h in (H, Hk, Hk, H))
    shape = B.make_shape(1, P, 0, 0, H, Hk, d, 0, 0.0, 0)
    table = np.asarray([(0, P, 0, 0), (P, small, 0, 1)], dtype=np.int32)
    tab = (shape, torch.from_numpy(table).cuda(), table, P + small)
    mk = lambda t: torch.full_like(t, float("nan"))   # noqa: E731
    o, dq, dk, dv = mk(q), mk(q), mk(k), mk(v)
    lse = torch.empty((H, P + small), device="cuda")
    ws = lambda op: torch.full((max(16, B.dualkv_groups_workspace_bytes(shape, 2, P + small, op)),), 0xFF, dtype=torch.uint8, device="cuda")   # noqa: E731
    B.dualkv_ctx_fwd_groups(*tab, q, k, v, o, lse, ws(B.OP_CTX_FWD))
    B.dualkv_ctx_bwd_groups(*tab, do, o, lse, q, k, v, dq, dk, dv, None, None, ws(B.OP_CTX_BWD))
    for lo, n in ((0, P), (P, small)):
        at = slice(lo, lo + n)
        s = B.make_shape(1, n, 0, 0, H, Hk, d, 0, 0.0, 0)
        one = torch.full((B.dualkv_workspace_bytes(s, B.OP_CTX_BWD),), 0xFF, dtype=torch.uint8, device="cuda")
        dq1, dk1, dv1 = mk(q[at]), mk(k[at]), mk(v[at])
        B.dualkv_ctx_bwd(s, do[at], o[at], lse[:, at].contiguous(), q[at], k[at], v[at], dq1, dk1, dv1, None, None, one)
        torch.cuda.synchronize()
        for got, want in ((dk[at], dk1), (dv[at], dv1), (dq[at], dq1)):
            assert not torch.isnan(want).any() and torch.equal(got.contiguous().view(torch.int16), want.view(torch.int16))
        G = H // Hk
        for hk in range(Hk):
            ek, ev = _exact(q[at, hk * G:(hk + 1) * G].double(), k[at, hk].double(), v[at, hk].double(),
                            do[at, hk * G:(hk + 1) * G].double(), d ** -0.5)
            # bf16 operands: 2^-8 each of P, dS and the result, in the 2-norm well below their sum
            for got, want in ((dk1[:, hk], ek), (dv1[:, hk], ev)):
                assert (got.double() - want).norm() <= 1e-2 * want.norm()
