"""GPU parity of dK/dV tiles whose row blocks are cut into parts for several workgroups (few key tiles, many row blocks and
heads): Call 2 (Call 1's are never cut) with the fp32 joint accumulation, against the fp64 oracle; parts that end inside a
sequence, empty sequences, a single sequence, groups of unequal prompts."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

import parity_util as PU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 96, 128, 192, 256, 512])
@pytest.mark.parametrize("P,lens", [(777, [130, 0, 97, 1]), (545, [515]), (31, [600, 33])])
def test_joint_accumulation_in_parts(d, P, lens):
    from paper_2605_15422_amd import binding as B
    print("case parts", d, P, lens, flush=True)
    shape = W.Shape("parts", len(lens), P, 0, 0, 8, 1, d, 0, seed=6000 + d + P)
    wl = W.make_workload(shape, resp_lens=np.asarray(lens))
    PU.bounded_parity(wl, flags=B.FLAG_ACCUM_CTX_F32)


@pytest.mark.parametrize("d", [64, 96, 128, 192, 256, 512])
@pytest.mark.parametrize("accum", [False, True])
def test_more_than_sixteen_parts(d, accum):
    """Sixty short sequences behind one key tile: thirty parts and more."""
    from paper_2605_15422_amd import binding as B
    print("case many parts", d, accum, flush=True)
    lens = [(7 * i) % 90 for i in range(60)]
    wl = W.make_workload(W.Shape("parts", len(lens), 31, 0, 0, 8, 1, d, 0, seed=6500 + d), resp_lens=np.asarray(lens))
    PU.bounded_parity(wl, flags=B.FLAG_ACCUM_CTX_F32 if accum else 0)


def test_groups_in_parts():
    """Seventy sequences in two groups (the search for a part's first sequence takes more than one 64-lane step)."""
    from oracle import attention_oracle as orc
    import torch
    from paper_2605_15422_amd import binding as B
    print("case groups in parts", flush=True)
    H, Hk, d = 4, 1, 64
    specs = [(300, [(5 * i) % 7 for i in range(67)]), (150, [90, 0, 40])]
    wls = [W.make_workload(W.Shape("g%d" % g, len(l), P, 0, 0, H, Hk, d, 0, seed=611 + g), resp_lens=np.asarray(l))
           for g, (P, l) in enumerate(specs)]
    cat = lambda n: torch.cat([B.bf16_from_bits(getattr(w, n)) for w in wls])   # noqa: E731
    t = {n: cat(n) for n in ("q_c", "k_c", "v_c", "do_c", "q_d", "k_d", "v_d", "do_d")}
    lens = np.concatenate([w.resp_lens for w in wls])
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    table = np.asarray([(0, 300, 0, 67), (300, 150, 67, 70)], dtype=np.int32)
    s = B.make_shape(70, 300, int(cu[-1]), int(lens.max()), H, Hk, d, 0, 0.0, B.FLAG_ACCUM_CTX_F32)
    gd, cud = torch.from_numpy(table).cuda(), torch.from_numpy(cu).cuda()
    ws = {op: torch.empty(max(16, B.dualkv_groups_workspace_bytes(s, 2, 450, op)), dtype=torch.uint8, device="cuda")
          for op in (B.OP_CTX_FWD, B.OP_FWD, B.OP_CTX_BWD, B.OP_BWD)}
    o_c, o_d, dq_c, dq_d = (torch.empty_like(t[n]) for n in ("q_c", "q_d", "q_c", "q_d"))
    dk_d, dv_d = torch.empty_like(t["k_d"]), torch.empty_like(t["v_d"])
    lse_c, lse_d = torch.empty((H, 450), device="cuda"), torch.empty((H, int(cu[-1])), device="cuda")
    acc = [torch.zeros((450, Hk, d), device="cuda") for _ in range(2)]
    B.dualkv_ctx_fwd_groups(s, gd, table, 450, t["q_c"], t["k_c"], t["v_c"], o_c, lse_c, ws[B.OP_CTX_FWD])
    B.dualkv_fwd_groups(s, gd, table, 450, t["q_d"], t["k_c"], t["v_c"], t["k_d"], t["v_d"], cud, cu, o_d, lse_d, ws[B.OP_FWD])
    B.dualkv_bwd_groups(s, gd, table, 450, t["do_d"], o_d, lse_d, t["q_d"], t["k_c"], t["v_c"], t["k_d"], t["v_d"], cud, cu,
                        dq_d, None, None, dk_d, dv_d, *acc, ws[B.OP_BWD])
    B.dualkv_ctx_bwd_groups(s, gd, table, 450, t["do_c"], o_c, lse_c, t["q_c"], t["k_c"], t["v_c"], dq_c, None, None, *acc,
                            ws[B.OP_CTX_BWD])
    torch.cuda.synchronize()
    c0 = r0 = 0
    for (P, _), wl in zip(specs, wls):
        x = PU.oracle_inputs(wl)
        ref = orc.dualkv_reference(x["q_c"], x["k_c"], x["v_c"], x["q_d"], x["k_d"], x["v_d"], wl.cu_seqlens, wl.scale,
                                   x["do_c"], x["do_d"], 0)
        T, rep = wl.total_resp, []
        PU.compare("dK_c", PU.to_f64(acc[0][c0:c0 + P]), ref["total"]["dk_c"], rep)
        PU.compare("dV_c", PU.to_f64(acc[1][c0:c0 + P]), ref["total"]["dv_c"], rep)
        PU.compare("dK_d", PU.to_f64(dk_d[r0:r0 + T]), ref["call2"]["dk_d"], rep)
        PU.compare("dQ_d", PU.to_f64(dq_d[r0:r0 + T]), ref["call2"]["dq_d"], rep)
        PU.compare("dQ_c", PU.to_f64(dq_c[c0:c0 + P]), ref["call1"]["dq_c"], rep)
        c0, r0 = c0 + P, r0 + T
