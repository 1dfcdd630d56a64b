"""GPU parity of the dK/dV kernel of which two workgroups share a CU (head dims 96 and 128, many prompt tiles; test_launch_rules.py
checks that these sizes go there): a last prompt tile of one key, responses around its 32-row blocks and 128-key tiles, empty ones,
whole tiles and tiles in parts that end inside a sequence, one to eight query heads per KV head, views of a packed projection; the
routes of a call with one group, of given row statistics and of sums that hold something already; the calls that the other
kernel takes; the largest token stride."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

import parity_util as PU

pytestmark = pytest.mark.gpu

SIZES = {"whole": (64, 32, 1537, [300, 129, 64, 33, 1, 0, 97, 31]), "parts": (8, 4, 4097, [301, 0, 515, 33, 250, 100]),
         "G1": (8, 8, 4097, [301, 0, 33, 200]), "G3": (12, 4, 9001, [100, 0, 33, 129]), "G4": (32, 8, 4097, [301, 0, 33, 200]),
         "G8": (32, 4, 8100, [65, 33, 100])}


@pytest.mark.parametrize("d", [96, 128])
@pytest.mark.parametrize("size", list(SIZES))
def test_pair(d, size):
    """Call 2 alone (its prompt gradients in the fp32 sums, too), every key of three KV heads."""
    import torch
    from oracle import attention_oracle as orc
    from paper_2605_15422_amd import binding as B, runner
    H, Hk, P, lens = SIZES[size]
    wl = W.make_workload(W.Shape("pair", len(lens), P, 0, 0, H, Hk, d, 0, seed=7300 + d), resp_lens=np.asarray(lens))
    x = PU.oracle_inputs(wl)
    keys = [(i, j) for i, R in enumerate(lens) for j in range(R)]
    want = {hk: orc.key_columns_call2(x["q_d"], x["k_c"], x["v_c"], x["k_d"], x["v_d"], wl.cu_seqlens, wl.scale, x["do_d"], hk,
                                      np.arange(P), keys) for hk in (0, 1, Hk - 1)}
    flags = B.FLAG_ACCUM_CTX_F32
    for mode in ("plain", "packed"):
        print("case pair", d, size, mode, flush=True)
        dg = B.upload(wl, flags)
        if mode == "packed":
            qkv = torch.cat([dg.q_d, dg.k_d, dg.v_d], dim=1)
            dg.q_d, dg.k_d, dg.v_d = qkv[:, :H], qkv[:, H:H + Hk], qkv[:, H + Hk:]
        b = runner.alloc(dg)
        runner.forward(dg, b, call1=False)
        runner.backward(dg, b, call1=False)
        torch.cuda.synchronize()
        rep = []
        for hk, (dk_c, dv_c, dk_d, dv_d) in want.items():
            PU.compare("dK_c", PU.to_f64(b.dk_c_acc[:, hk]), dk_c, rep)
            PU.compare("dV_c", PU.to_f64(b.dv_c_acc[:, hk]), dv_c, rep)
            PU.compare("dK_d", PU.to_f64(b.dk_d[:, hk]), dk_d, rep)
            PU.compare("dV_d", PU.to_f64(b.dv_d[:, hk]), dv_d, rep)
        print("\n".join(rep), flush=True)


def _group(d, size, flags):
    from paper_2605_15422_amd import binding as B, runner
    H, Hk, P, lens = SIZES[size]
    dg = B.upload(W.make_workload(W.Shape("pair", len(lens), P, 0, 0, H, Hk, d, 0, seed=7400 + d), resp_lens=np.asarray(lens)), flags)
    b = runner.alloc(dg)
    runner.forward(dg, b, call1=False)
    return dg, b


def _backward(dg, b, skip=0, dq=None):
    """Call 2's backward with fresh outputs and sums: (dk_c, dv_c sums, dk_d, dv_d)."""
    import torch
    from paper_2605_15422_amd import binding as B
    s = type(dg.shape_c).from_buffer_copy(bytes(dg.shape_c))
    s.flags |= skip
    acc = [torch.zeros(dg.k_c.shape, dtype=torch.float32, device="cuda") for _ in range(2)]
    out = [torch.full(dg.k_d.shape, float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    B.dualkv_bwd(s, dg.do_d, b.o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d, dg.cu_dev, dg.cu_host, b.dq_d if dq is None else dq,
                 None, None, *out, *acc, b.ws_bwd)
    torch.cuda.synchronize()
    return (*acc, *out)


# (tiles in one part: every sum has one term, and all routes give the same bits)
@pytest.mark.parametrize("d", [96, 128])
def test_pair_routes(d):
    import torch
    from paper_2605_15422_amd import binding as B
    dg, b = _group(d, "G1", B.FLAG_ACCUM_CTX_F32)
    want = _backward(dg, b)

    def check(route, got):
        print("case pair route", d, route, flush=True)
        for x, y in zip(got, want):
            assert not torch.isnan(x).any() and torch.equal(x, y), route

    # statistics of an earlier call: from the dQ kernel, then from the preprocess (the dQ stage alone runs it by itself)
    for first in (B.FLAG_SKIP_DKDV, B.FLAG_SKIP_DKDV | B.FLAG_SKIP_DQ):
        b.ws_bwd.fill_(0xFF)
        _backward(dg, b, first)
        check("given statistics", _backward(dg, b, B.FLAG_SKIP_PRE | B.FLAG_SKIP_DQ))
    b.ws_bwd.fill_(0xFF)
    check("no dQ", _backward(dg, b, B.FLAG_SKIP_DQ))
    # dQ over Q: written last
    q = dg.q_d.clone()
    b.ws_bwd.fill_(0xFF)
    check("dQ over Q", _backward(dg, b, dq=dg.q_d))
    assert torch.equal(dg.q_d, b.dq_d)
    dg.q_d.copy_(q)

    # sums that hold something: one addition to each
    acc = [torch.randn(dg.k_c.shape, device="cuda") for _ in range(2)]
    start = [x.clone() for x in acc]
    out = [torch.empty_like(dg.k_d) for _ in range(2)]
    args = (dg.do_d, b.o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d, dg.cu_dev, dg.cu_host, b.dq_d, None, None, *out, *acc)
    B.dualkv_bwd(dg.shape_c, *args, b.ws_bwd)
    torch.cuda.synchronize()
    for x, x0, w in zip(acc, start, want):
        assert torch.equal(x, x0 + w)

    # a *_groups call with one group
    N, P = dg.shape_c.n_seqs, dg.shape_c.ctx_len
    table = np.asarray([(0, P, 0, N)], dtype=np.int32)
    ws = torch.full((B.dualkv_groups_workspace_bytes(dg.shape_c, 1, P, B.OP_BWD),), 0xFF, dtype=torch.uint8, device="cuda")
    for x in acc:
        x.zero_()
    B.dualkv_bwd_groups(dg.shape_c, torch.from_numpy(table).cuda(), table, P, *args, ws)
    torch.cuda.synchronize()
    check("one group", (*acc, *out))


# dkdv4 takes the same work without the joint sums, and with a second group beside it; both sides round sums in another order to bf16, half
# a unit (2^-9) each
@pytest.mark.parametrize("d", [96, 128])
def test_pair_and_other_kernel_agree(d):
    import torch
    from paper_2605_15422_amd import binding as B
    print("case pair other kernel", d, flush=True)
    dg, b = _group(d, "G1", B.FLAG_ACCUM_CTX_F32)
    want = _backward(dg, b)

    def check(got):
        for x, y in zip(got, want):
            assert (x.double() - y.double()).norm() <= 2.0**-8 * y.double().norm()

    two = type(dg.shape_c).from_buffer_copy(bytes(dg.shape_c))
    two.flags = 0
    out = [torch.empty_like(x) for x in (dg.k_c, dg.k_c, dg.k_d, dg.k_d)]
    ws = torch.full((B.dualkv_workspace_bytes(two, B.OP_BWD),), 0xFF, dtype=torch.uint8, device="cuda")
    B.dualkv_bwd(two, dg.do_d, b.o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d, dg.cu_dev, dg.cu_host, b.dq_d, *out, None, None, ws)
    torch.cuda.synchronize()
    check(out)

    # the group twice
    N, P, T = dg.shape_c.n_seqs, dg.shape_c.ctx_len, dg.shape_c.total_resp
    table = np.asarray([(0, P, 0, N), (P, P, N, 2 * N)], dtype=np.int32)
    cu = np.concatenate([dg.cu_host, dg.cu_host[1:] + T]).astype(np.int32)
    both = type(dg.shape_c).from_buffer_copy(bytes(dg.shape_c))
    both.n_seqs, both.total_resp = 2 * N, 2 * T

    def twice(x):
        return torch.cat([x, x])

    acc = [torch.zeros((2 * P, *dg.k_c.shape[1:]), dtype=torch.float32, device="cuda") for _ in range(2)]
    out = [torch.empty_like(twice(dg.k_d)) for _ in range(2)]
    ws = torch.full((B.dualkv_groups_workspace_bytes(both, 2, 2 * P, B.OP_BWD),), 0xFF, dtype=torch.uint8, device="cuda")
    B.dualkv_bwd_groups(both, torch.from_numpy(table).cuda(), table, 2 * P, *(twice(x) for x in (dg.do_d, b.o_d)), torch.cat([b.lse_d] * 2, dim=1).contiguous(),
                        *(twice(x) for x in (dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d)), torch.from_numpy(cu).cuda(), cu, torch.empty_like(twice(b.dq_d)), None, None,
                        *out, *acc, ws)
    torch.cuda.synchronize()
    for g in range(2):
        check([x[g * P:(g + 1) * P] for x in acc] + [x[g * T:(g + 1) * T] for x in out])


@pytest.mark.parametrize("d", [96, 128])
def test_pair_largest_token_stride(d):
    """Q, dO and the response K, V as views whose token stride is the documented maximum (2^22 elements)."""
    import torch
    from paper_2605_15422_amd import binding as B
    print("case pair max_stride", d, flush=True)
    dg, b = _group(d, "G1", B.FLAG_ACCUM_CTX_F32)
    want = _backward(dg, b)
    TS, T, H = 1 << 22, dg.q_d.shape[0], dg.q_d.shape[1]
    big = torch.empty(T * TS, dtype=torch.bfloat16, device="cuda")
    names = ("q_d", "do_d", "k_d", "v_d")
    views = [big.as_strided((T, H, d), (TS, d, 1), i * H * d) for i in range(len(names))]
    for n, v in zip(names, views):
        v.copy_(getattr(dg, n))
    for n, v in zip(names, views):
        setattr(dg, n, v)
    out = [torch.empty((T, H, d), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    acc = [torch.zeros(dg.k_c.shape, dtype=torch.float32, device="cuda") for _ in range(2)]
    dq = torch.empty_like(b.dq_d)
    B.dualkv_bwd(dg.shape_c, dg.do_d, b.o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d, dg.cu_dev, dg.cu_host, dq, None, None, *out, *acc,
                 b.ws_bwd)
    torch.cuda.synchronize()
    assert torch.equal(dq, b.dq_d)
    for x, y in zip((*acc, *out), want):
        assert torch.equal(x, y)
