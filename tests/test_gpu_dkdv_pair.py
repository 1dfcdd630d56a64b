"""GPU parity of the dK/dV kernel of which two workgroups share a CU (head dims 96 and 128, many prompt tiles; test_launch_rules.py
checks that these sizes go there): a last prompt tile of one key, responses around its 32-row blocks and 128-key tiles, empty ones,
whole tiles and tiles in three parts that end inside a sequence, views of a packed projection."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

import parity_util as PU

pytestmark = pytest.mark.gpu

SIZES = {"whole": (64, 32, 1537, [300, 129, 64, 33, 1, 0, 97, 31]), "parts": (8, 4, 4097, [301, 0, 515, 33, 250, 100])}


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
