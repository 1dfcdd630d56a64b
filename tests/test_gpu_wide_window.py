"""A window at the end of its type's range sees what a window over all positions sees, forward and backward, in both calls."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 96, 128, 192, 256])
def test_widest_window(d):
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case widest window", d, flush=True)
    lens, P, out = [70, 0, 333, 1], 200, []
    for window in (P + max(lens), 2**31 - 1):
        dg = B.upload(W.make_workload(W.Shape("wide", len(lens), P, 0, 0, 4, 2, d, window, seed=5), resp_lens=np.asarray(lens)))
        b = runner.alloc(dg)
        runner.layer_step(dg, b)
        torch.cuda.synchronize()
        out.append([getattr(b, k) for k in ("o_c", "o_d", "dq_c", "dq_d", "dk_c1", "dv_c1", "dk_d", "dv_d", "dk_c2", "dv_c2")])
    for i, (x, y) in enumerate(zip(*out)):
        if i < 8:
            assert not torch.isnan(x).any() and torch.equal(x.view(torch.int16), y.view(torch.int16))
        else:   # (the parts of a prompt tile add in any order: one rounding of fp32 sums to bf16)
            assert (x.double() - y.double()).norm() <= 2.0**-8 * y.double().norm()
