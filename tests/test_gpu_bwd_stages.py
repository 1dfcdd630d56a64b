"""The backward calls form D = rowsum(dO * O) inside the dQ kernel; with DUALKV_FLAG_SKIP_DQ, or when dQ overwrites an input
of the dK/dV kernel, a preprocess kernel does, bit for bit alike.  Both routes against the fp64 oracle, every head dim, partial row blocks."""
import numpy as np
import pytest

from oracle import attention_oracle as orc
from paper_2605_15422_amd import workloads as W

import parity_util as PU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 96, 128, 192, 256, 512])
@pytest.mark.parametrize("route", ["stages", "in_place_do", "in_place_o"])
def test_bwd_routes(d, route):
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case", route, d, flush=True)
    shape = W.Shape("routes", 3, 75, 0, 0, 4, 2, d, 0, seed=31 + d)
    wl = W.make_workload(shape, resp_lens=np.asarray([33, 1, 70]))
    x = PU.oracle_inputs(wl)
    ref = orc.dualkv_reference(x["q_c"], x["k_c"], x["v_c"], x["q_d"], x["k_d"], x["v_d"], wl.cu_seqlens, wl.scale,
                               x["do_c"], x["do_d"], 0)
    dg = B.upload(wl)
    b = runner.alloc(dg)
    runner.forward(dg, b)

    def bwd(flags, o_d, do_d, dq_d, o_c, do_c, dq_c):
        s = type(dg.shape_c).from_buffer_copy(bytes(dg.shape_c))
        s.flags = flags
        B.dualkv_bwd(s, do_d, o_d, b.lse_d, dg.q_d, dg.k_c, dg.v_c, dg.k_d, dg.v_d, dg.cu_dev, dg.cu_host, dq_d, b.dk_c2,
                     b.dv_c2, b.dk_d, b.dv_d, None, None, b.ws_bwd)
        B.dualkv_ctx_bwd(s, do_c, o_c, b.lse_c, dg.q_c, dg.k_c, dg.v_c, dq_c, b.dk_c1, b.dv_c1, None, None, b.ws_ctx_bwd)

    plain = (b.o_d, dg.do_d, b.dq_d, b.o_c, dg.do_c, b.dq_c)
    if route == "stages":
        bwd(B.FLAG_SKIP_DQ | B.FLAG_SKIP_DKDV, *plain)
        bwd(B.FLAG_SKIP_PRE | B.FLAG_SKIP_DKDV, *plain)
        bwd(B.FLAG_SKIP_PRE | B.FLAG_SKIP_DQ, *plain)
        dq_d, dq_c = b.dq_d, b.dq_c
    elif route == "in_place_do":
        dq_d, dq_c = dg.do_d.clone(), dg.do_c.clone()
        bwd(0, b.o_d, dq_d, dq_d, b.o_c, dq_c, dq_c)
    else:
        dq_d, dq_c = b.o_d.clone(), b.o_c.clone()
        bwd(0, dq_d, dg.do_d, dq_d, dq_c, dg.do_c, dq_c)
    got_dq = [t.clone() for t in (dq_d, dq_c)]
    kept = [t.clone() for t in (b.dk_d, b.dv_d)]
    bwd(0, *plain)
    torch.cuda.synchronize()
    for a, c in zip(got_dq + kept, (b.dq_d, b.dq_c, b.dk_d, b.dv_d)):
        assert torch.equal(a.view(torch.int16), c.view(torch.int16))
    rep = []
    for n, got, want in (("dQ_d", dq_d, ref["call2"]["dq_d"]), ("dK_d", b.dk_d, ref["call2"]["dk_d"]),
                         ("dV_d", b.dv_d, ref["call2"]["dv_d"]), ("dK_c2", b.dk_c2, ref["call2"]["dk_c"]),
                         ("dV_c2", b.dv_c2, ref["call2"]["dv_c"]), ("dQ_c", dq_c, ref["call1"]["dq_c"]),
                         ("dK_c1", b.dk_c1, ref["call1"]["dk_c"]), ("dV_c1", b.dv_c1, ref["call1"]["dv_c"])):
        PU.compare(n, PU.to_f64(got), want, rep)
