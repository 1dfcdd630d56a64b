"""Forward and dQ of head dims 64 to 128 in workgroups of four waves (K and V tiles travel in halves of 32 keys in the forward kernel, V
one tile ahead in dQ) at the edges of halves and tiles of both regions, and the calls that go to eight waves instead."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

import parity_util as PU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("P", [1, 33, 96, 161])
@pytest.mark.parametrize("window", [0, 40])
def test_edges_of_halves(d, P, window):
    print("case halves", d, P, window, flush=True)
    lens = [1, 32, 33, 64, 0, 97, 130] * 10   # (enough row blocks for workgroups that share a CU)
    shape = W.Shape("halves", len(lens), P, 0, 0, 16, 4, d, window, seed=130 + d + P)
    PU.bounded_parity(W.make_workload(shape, resp_lens=np.asarray(lens)))


@pytest.mark.parametrize("d,H,Hk,P", [(64, 32, 8, 3393), (96, 32, 8, 3340), (96, 8, 8, 13569), (128, 32, 8, 3393), (128, 8, 2, 16384)])
def test_one_causal_sequence_as_two_groups(d, H, Hk, P):
    """One prompt in two rounds of eight waves, and twice in one call of two groups, which takes four: a row's tiles, their order and
    its arithmetic are the same, so are its bits."""
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case two groups", d, H, Hk, P, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(d + P)
    q, k, v, do = (torch.randn((P, h, d), generator=gen, device="cuda").bfloat16() for h in (H, Hk, Hk, H))
    shape = B.make_shape(1, P, 0, 0, H, Hk, d, 0, 0.0, 0)
    table = np.asarray([(0, P, 0, 0), (P, P, 0, 1)], dtype=np.int32)
    dev = torch.from_numpy(table).cuda()
    ws = lambda op: torch.full((max(16, B.dualkv_groups_workspace_bytes(shape, 2, 2 * P, op)),), 0xFF, dtype=torch.uint8, device="cuda")   # noqa: E731
    two = lambda x: torch.cat([x, x])   # noqa: E731
    o1, dq1 = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    o2, dq2 = two(o1), two(dq1)
    l1, l2 = torch.empty((H, P), device="cuda"), torch.empty((H, 2 * P), device="cuda")
    g1, g2 = [torch.empty_like(k) for _ in range(2)], [torch.empty_like(two(k)) for _ in range(2)]
    B.dualkv_ctx_fwd(shape, q, k, v, o1, l1)
    one = torch.full((B.dualkv_workspace_bytes(shape, B.OP_CTX_BWD),), 0xFF, dtype=torch.uint8, device="cuda")
    B.dualkv_ctx_bwd(shape, do, o1, l1, q, k, v, dq1, *g1, None, None, one)
    tab = (shape, dev, table, 2 * P)
    B.dualkv_ctx_fwd_groups(*tab, two(q), two(k), two(v), o2, l2, ws(B.OP_CTX_FWD))
    B.dualkv_ctx_bwd_groups(*tab, two(do), o2, l2, two(q), two(k), two(v), dq2, *g2, None, None, ws(B.OP_CTX_BWD))
    torch.cuda.synchronize()
    bits = lambda x: x.view(torch.int16) if x.dtype == torch.bfloat16 else x.view(torch.int32)   # noqa: E731
    for half in (slice(0, P), slice(P, 2 * P)):
        assert not torch.isnan(o1).any() and torch.equal(bits(o1), bits(o2[half]))
        assert not torch.isnan(dq1).any() and torch.equal(bits(dq1), bits(dq2[half]))
        assert torch.equal(bits(l1), bits(l2[:, half].contiguous()))
        for a, b in zip(g1, g2):
            assert torch.equal(bits(a), bits(b[half]))
