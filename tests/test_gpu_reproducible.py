"""Sums of the prompt gradients that have one order have one result: Call 1 adds to every element of the fp32 joint
accumulators once, so that a joint sum of Call 1 alone is the two-term result before its cast; Call 2 adds to zeroed ones at
most twice where its prompt tiles have at most two parts."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,Hk,P", [(64, 8, 1, 2048), (96, 8, 1, 1500), (128, 32, 1, 1024), (128, 8, 2, 3000), (192, 8, 1, 1000),
                                      (256, 8, 1, 1000), (512, 8, 1, 700)])
def test_call1_joint_sum_is_the_two_term_sum(d, H, Hk, P):
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case call 1 joint", d, H, Hk, P, flush=True)
    dg = B.upload(W.make_workload(W.Shape("joint", 1, P, 0, 0, H, Hk, d, 0, seed=700 + d), resp_lens=np.asarray([0])))
    b = runner.alloc(dg)
    runner.forward(dg, b, call2=False)
    runner.backward(dg, b, call2=False)
    s = type(dg.shape_c).from_buffer_copy(bytes(dg.shape_c))
    s.flags = B.FLAG_ACCUM_CTX_F32
    for _ in range(2):
        acc = [torch.zeros((P, Hk, d), device="cuda") for _ in range(2)]
        B.dualkv_ctx_bwd(s, dg.do_c, b.o_c, b.lse_c, dg.q_c, dg.k_c, dg.v_c, b.dq_c, None, None, *acc, b.ws_ctx_bwd)
        B.dualkv_finalize_ctx_grads(s, *acc, b.dk_c2, b.dv_c2)
        torch.cuda.synchronize()
        assert torch.equal(b.dk_c2, b.dk_c1) and torch.equal(b.dv_c2, b.dv_c1)


@pytest.mark.parametrize("d,H,Hk,P,lens", [(64, 8, 1, 700, [900, 800]), (96, 8, 2, 1500, [700, 30]), (128, 32, 4, 86, [1900, 719]),
                                           (128, 16, 8, 5000, [300, 200, 100, 400]), (192, 8, 2, 600, [1000]), (256, 8, 2, 1200, [800, 500]),
                                           (512, 8, 1, 500, [400, 300])])
@pytest.mark.parametrize("joint", [False, True])
def test_two_parts_have_one_sum(d, H, Hk, P, lens, joint):
    """Call 2 with one or two parts a prompt tile: the same bits from run to run, whichever part adds first."""
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case two parts", d, H, Hk, P, joint, flush=True)
    dg = B.upload(W.make_workload(W.Shape("two", len(lens), P, 0, 0, H, Hk, d, 0, seed=800 + d), resp_lens=np.asarray(lens)),
                  B.FLAG_ACCUM_CTX_F32 if joint else 0)
    b = runner.alloc(dg)
    want = None
    for _ in range(6):
        runner.layer_step(dg, b)
        torch.cuda.synchronize()
        got = [t.clone() for t in ((b.dk_c_acc, b.dv_c_acc) if joint else (b.dk_c2, b.dv_c2))]
        want = want or got
        for x, y in zip(got, want):
            assert torch.equal(x, y)
