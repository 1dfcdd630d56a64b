"""Backward calls with few workgroups run dK/dV and dQ in one launch: bit for bit what the two kernels give in launches of
their own, on both sides of the limits, around the 32-row and 128-key tiles, with a window, an empty response and
several head counts."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

import parity_util as PU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("H,Hk,P,lens", [(2, 1, 1, [1]), (4, 2, 128, [33, 0, 129]), (8, 8, 1021, [128, 32, 31]), (16, 4, 1500, [300] * 4),
                                         (32, 8, 130, [64] * 8), (32, 8, 130, [200] * 12), (8, 2, 700, [300, 1, 523]),
                                         (8, 2, 300, [700] * 5 + [90]), (6, 1, 0, [257, 5])])
@pytest.mark.parametrize("window", [0, 70])
def test_together_as_apart(d, H, Hk, P, lens, window):
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case together", d, H, Hk, P, len(lens), window, flush=True)
    dg = B.upload(W.make_workload(W.Shape("together", len(lens), P, 0, 0, H, Hk, d, window, seed=90 + d), resp_lens=np.asarray(lens)))
    out = []
    for flags in ((0,), (B.FLAG_SKIP_DKDV, B.FLAG_SKIP_PRE | B.FLAG_SKIP_DQ)):
        b = runner.alloc(dg)
        runner.forward(dg, b, call1=P > 0)
        for f in flags:
            s = type(dg.shape_c).from_buffer_copy(bytes(dg.shape_c))
            s.flags = f
            B.dualkv_bwd(s, dg.do_d, b.o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d, dg.cu_dev, dg.cu_host, b.dq_d,
                         b.dk_c2, b.dv_c2, b.dk_d, b.dv_d, None, None, b.ws_bwd)
            if P:
                B.dualkv_ctx_bwd(s, dg.do_c, b.o_c, b.lse_c, dg.q_c, dg.k_c, dg.v_c, b.dq_c, b.dk_c1, b.dv_c1, None, None,
                                 b.ws_ctx_bwd)
        torch.cuda.synchronize()
        out.append([b.dq_d, b.dk_d, b.dv_d] + ([b.dq_c, b.dk_c1, b.dv_c1] if P else []))
    for x, y in zip(*out):
        assert not torch.isnan(x).any() and torch.equal(x.view(torch.int16), y.view(torch.int16))


# 256 to 640 workgroups: more than one a CU
SHARED = [(32, 8, 130, [64] * 8), (16, 4, 700, [300] * 4), (8, 2, 300, [400] * 5 + [90])]


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("H,Hk,P,lens", SHARED)
@pytest.mark.parametrize("accum", [False, True])
def test_prompt_gradients_of_a_shared_launch(d, H, Hk, P, lens, accum):
    """The prompt tiles come first, in parts that add to cleared accumulators: every gradient within its rounding bound."""
    from paper_2605_15422_amd import binding as B
    print("case shared", d, H, Hk, P, len(lens), accum, flush=True)
    wl = W.make_workload(W.Shape("shared", len(lens), P, 0, 0, H, Hk, d, 0, seed=120 + d), resp_lens=np.asarray(lens))
    PU.bounded_parity(wl, B.FLAG_ACCUM_CTX_F32 if accum else 0)


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("H,Hk,P,lens", SHARED)
def test_prompt_gradients_together_as_apart(d, H, Hk, P, lens):
    """One launch may cut a prompt tile into other parts than two launches do: fp32 sums in another order (a part of the sum at
    2^-24 each, far below the tolerance), then one rounding to bf16 (2^-9 of an element)."""
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case prompt together", d, H, Hk, P, len(lens), flush=True)
    dg = B.upload(W.make_workload(W.Shape("together", len(lens), P, 0, 0, H, Hk, d, 0, seed=90 + d), resp_lens=np.asarray(lens)))
    out = []
    for flags in ((0,), (B.FLAG_SKIP_DKDV, B.FLAG_SKIP_PRE | B.FLAG_SKIP_DQ)):
        b = runner.alloc(dg)
        runner.forward(dg, b)
        for f in flags:
            s = type(dg.shape_c).from_buffer_copy(bytes(dg.shape_c))
            s.flags = f
            B.dualkv_bwd(s, dg.do_d, b.o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d, dg.cu_dev, dg.cu_host, b.dq_d,
                         b.dk_c2, b.dv_c2, b.dk_d, b.dv_d, None, None, b.ws_bwd)
        torch.cuda.synchronize()
        out.append([b.dk_c2.double(), b.dv_c2.double()])
    for x, y in zip(*out):
        assert (x - y).norm() <= 2.0**-9 * y.norm()
