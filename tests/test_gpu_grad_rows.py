"""Rows of dK and dV: tiles that end inside a key tile write their own rows and nothing else, whatever the strides, and add to
their own elements of the fp32 sums."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

pytestmark = pytest.mark.gpu

MARK = 0x7F55   # a NaN that no kernel writes


def _strided(t, kind):
    """An output of t's shape inside a marked buffer: heads apart, or head-major; and the buffer."""
    import torch
    rows, heads, d = t.shape
    if kind == "apart":
        buf = torch.full((rows + 150, heads + 1, d + 24), MARK, dtype=torch.int16, device="cuda")
        return buf.view(torch.bfloat16)[3:3 + rows, :heads, 8:8 + d], buf
    buf = torch.full((heads + 1, rows + 150, d), MARK, dtype=torch.int16, device="cuda")
    return buf.view(torch.bfloat16)[:heads, 3:3 + rows].transpose(0, 1), buf


@pytest.mark.parametrize("d", [64, 96, 128, 192, 256, 512])
@pytest.mark.parametrize("kind", ["apart", "head-major"])
def test_gradient_rows_end_where_their_tile_ends(d, kind):
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case rows", d, kind, flush=True)
    lens, P = [1, 31, 33, 64, 0, 65, 127, 129], 161
    dg = B.upload(W.make_workload(W.Shape("rows", len(lens), P, 0, 0, 4, 2, d, 0, seed=300 + d), resp_lens=np.asarray(lens)))
    b = runner.alloc(dg)
    runner.layer_step(dg, b)
    s = dg.shape_c
    outs = {n: _strided(getattr(b, n), kind) for n in ("dk_d", "dv_d", "dk_c1", "dv_c1")}
    B.dualkv_bwd(s, dg.do_d, b.o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d, dg.cu_dev, dg.cu_host, b.dq_d, b.dk_c2, b.dv_c2,
                 outs["dk_d"][0], outs["dv_d"][0], None, None, b.ws_bwd)
    B.dualkv_ctx_bwd(s, dg.do_c, b.o_c, b.lse_c, dg.q_c, dg.k_c, dg.v_c, b.dq_c, outs["dk_c1"][0], outs["dv_c1"][0], None, None, b.ws_ctx_bwd)
    torch.cuda.synchronize()
    for n, (view, buf) in outs.items():
        assert torch.equal(view.contiguous().view(torch.int16), getattr(b, n).view(torch.int16)), n
        view.view(torch.int16).fill_(MARK)
        assert (buf == MARK).all(), n


@pytest.mark.parametrize("d", [64, 96, 128, 192, 256, 512])
def test_sums_end_where_the_prompt_ends(d):
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case sums", d, flush=True)
    P, Hk = 161, 2
    dg = B.upload(W.make_workload(W.Shape("sums", 1, P, 0, 0, 4, Hk, d, 0, seed=320 + d), resp_lens=np.asarray([0])))
    b = runner.alloc(dg)
    runner.forward(dg, b, call2=False)
    runner.backward(dg, b, call2=False)
    s = type(dg.shape_c).from_buffer_copy(bytes(dg.shape_c))
    s.flags = B.FLAG_ACCUM_CTX_F32
    bufs = [torch.full((P + 150, Hk, d), 7.0, device="cuda") for _ in range(2)]
    for x in bufs:
        x[:P] = 0
    B.dualkv_ctx_bwd(s, dg.do_c, b.o_c, b.lse_c, dg.q_c, dg.k_c, dg.v_c, b.dq_c, None, None, bufs[0][:P], bufs[1][:P], b.ws_ctx_bwd)
    torch.cuda.synchronize()
    for x, want in zip(bufs, (b.dk_c1, b.dv_c1)):
        assert (x[P:] == 7.0).all() and torch.equal(x[:P].bfloat16(), want)
