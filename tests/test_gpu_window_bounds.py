"""Head dims 64 to 128 with windows around the places where a lane's bounds end: single keys, the four and sixteen keys of a score tile,
half tiles and tiles of 32 and 64 keys; rows whose first half tile holds no visible key, rows that see prompt and response."""
import numpy as np
import pytest

import parity_util as PU
from oracle import attention_oracle as orc
from paper_2605_15422_amd import runner, workloads as W
from paper_2605_15422_amd import binding as B

pytestmark = pytest.mark.gpu


def _workload(d, H, Hk, window):
    print("case window bounds", d, window, flush=True)
    lens = np.asarray([5, 0, 40, 131])
    return W.make_workload(W.Shape("bounds", len(lens), 75, 0, 0, H, Hk, d, window, seed=8100 + d + window), resp_lens=lens)


@pytest.mark.parametrize("d,H,Hk", [(64, 8, 2), (96, 4, 4), (128, 8, 2)])
@pytest.mark.parametrize("window", [1, 2, 4, 5, 15, 16, 17, 20, 31, 33, 63, 64, 65, 127, 200])
def test_window_bounds(d, H, Hk, window):
    import torch
    wl = _workload(d, H, Hk, window)
    x = PU.oracle_inputs(wl)
    ref = orc.dualkv_forward(x["q_c"], x["k_c"], x["v_c"], x["q_d"], x["k_d"], x["v_d"], wl.cu_seqlens, wl.scale, window)
    dg = B.upload(wl, 0)
    b = runner.alloc(dg)
    runner.forward(dg, b)
    torch.cuda.synchronize()
    rep = []
    for part, o, lse in (("c", b.o_c, b.lse_c), ("d", b.o_d, b.lse_d)):
        PU.compare("O_" + part, PU.to_f64(o), ref["o_" + part], rep)
        PU.compare_lse("LSE_" + part, PU.to_f64(lse), ref["lse_" + part], rep)
    print("\n".join(rep), flush=True)


# (with a window of one key, dQ and dK are zero)
@pytest.mark.parametrize("d,H,Hk", [(64, 8, 2), (96, 4, 4), (128, 8, 2)])
@pytest.mark.parametrize("window", [2, 5, 16, 17, 33, 65, 200])
def test_window_bounds_backward(d, H, Hk, window):
    PU.bounded_parity(_workload(d, H, Hk, window))
