"""dQ beside dK/dV in one launch past one workgroup a CU: one causal sequence (head dims 64 to 128 with dQ workgroups of four and of eight
waves), rows behind a prompt with dQ first and last.  Bit for bit what the two kernels give in launches of their own (prompt gradients: sums of
parts, to rounding)."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

pytestmark = pytest.mark.gpu


def _apart(s, run):
    from paper_2605_15422_amd import binding as B
    out = []
    for flags in ((0,), (B.FLAG_SKIP_DKDV, B.FLAG_SKIP_PRE | B.FLAG_SKIP_DQ)):
        out.append(run([type(s).from_buffer_copy(bytes(s)) for _ in flags], flags))
    return out


CAUSAL = [(d, *x) for d in (64, 96, 128) for x in ((16, 4, 2081), (8, 8, 2500), (32, 8, 3873), (8, 2, 16350), (32, 8, 6657))] + [
    (192, 2, 1, 65), (192, 8, 2, 3001), (192, 4, 4, 9600), (192, 16, 2, 2735), (256, 6, 2, 1023), (256, 8, 2, 4097), (256, 4, 4, 9700),
    (512, 2, 2, 31), (512, 8, 2, 2049), (512, 6, 2, 1500), (512, 4, 2, 9700)]


@pytest.mark.parametrize("d,H,Hk,P", CAUSAL)
def test_one_causal_sequence(d, H, Hk, P):
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case causal beside", d, H, Hk, P, flush=True)
    dg = B.upload(W.make_workload(W.Shape("beside", 1, P, 0, 0, H, Hk, d, 0, seed=400 + d), resp_lens=np.asarray([0])))
    b = runner.alloc(dg)
    runner.forward(dg, b, call2=False)

    def run(shapes, flags):
        o = [torch.full_like(x, float("nan")) for x in (dg.q_c, dg.k_c, dg.v_c)]
        b.ws_ctx_bwd.fill_(0xFF)
        for s, f in zip(shapes, flags):
            s.flags = f
            B.dualkv_ctx_bwd(s, dg.do_c, b.o_c, b.lse_c, dg.q_c, dg.k_c, dg.v_c, *o, None, None, b.ws_ctx_bwd)
        torch.cuda.synchronize()
        return o
    for x, y in zip(*_apart(dg.shape_c, run)):
        assert not torch.isnan(x).any() and torch.equal(x.view(torch.int16), y.view(torch.int16))


ROWS = [(d, *x) for d in (64, 96, 128) for x in ((32, 8, 4300, [20, 33]), (12, 4, 9000, [0, 1, 130]), (8, 8, 4097, [64] * 7), (32, 4, 8321, [97]))] + [
    (d, *x) for d in (192, 256, 512) for x in ((8, 2, 3001, [20, 0, 33]), (12, 4, 70, [700, 650, 31]), (4, 4, 500, [129] * 9), (8, 1, 1, [1, 64]))]


@pytest.mark.parametrize("d,H,Hk,P,lens", ROWS)
def test_rows_behind_a_prompt(d, H, Hk, P, lens):
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case dQ first", d, H, Hk, P, lens, flush=True)
    dg = B.upload(W.make_workload(W.Shape("first", len(lens), P, 0, 0, H, Hk, d, 0, seed=500 + d), resp_lens=np.asarray(lens)))
    b = runner.alloc(dg)
    runner.forward(dg, b, call1=False)

    def run(shapes, flags):
        o = [torch.full_like(x, float("nan")) for x in (dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d)]
        b.ws_bwd.fill_(0xFF)
        for s, f in zip(shapes, flags):
            s.flags = f
            B.dualkv_bwd(s, dg.do_d, b.o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d, dg.cu_dev, dg.cu_host, *o, None, None, b.ws_bwd)
        torch.cuda.synchronize()
        return o
    one, two = _apart(dg.shape_c, run)
    for k, (x, y) in enumerate(zip(one, two)):
        assert not torch.isnan(x).any()
        # (fp32 sums in another order, one rounding to bf16)
        if k in (1, 2): assert (x.double() - y.double()).norm() <= 2.0**-9 * y.double().norm()
        else: assert torch.equal(x.view(torch.int16), y.view(torch.int16))


@pytest.mark.parametrize("d,H,Hk,P,lens", [(128, 16, 4, 1000, []), (64, 8, 2, 300, [500, 31, 200]), (96, 32, 8, 4300, [20, 33]), (256, 8, 2, 900, []),
                                           (512, 8, 2, 600, [64, 33])])
def test_gradients_over_the_keys(d, H, Hk, P, lens):
    """dK and dV written over K and V: dQ is done by then."""
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case in place", d, H, Hk, P, lens, flush=True)
    dg = B.upload(W.make_workload(W.Shape("inplace", max(len(lens), 1), P, 0, 0, H, Hk, d, 0, seed=600 + d), resp_lens=np.asarray(lens or [0])))
    b = runner.alloc(dg)
    runner.layer_step(dg, b)
    s = dg.shape_c
    if lens:
        k, v = dg.k_d.clone(), dg.v_d.clone()
        dq = torch.full_like(dg.q_d, float("nan"))
        B.dualkv_bwd(s, dg.do_d, b.o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, k, v, dg.cu_dev, dg.cu_host, dq, b.dk_c2, b.dv_c2, k, v, None, None, b.ws_bwd)
        want = (b.dq_d, b.dk_d, b.dv_d)
    else:
        k, v = dg.k_c.clone(), dg.v_c.clone()
        dq = torch.full_like(dg.q_c, float("nan"))
        B.dualkv_ctx_bwd(s, dg.do_c, b.o_c, b.lse_c, dg.q_c, k, v, dq, k, v, None, None, b.ws_ctx_bwd)
        want = (b.dq_c, b.dk_c1, b.dv_c1)
    torch.cuda.synchronize()
    for x, y in zip((dq, k, v), want):
        assert torch.equal(x.view(torch.int16), y.view(torch.int16))
