"""Calls whose row blocks or key tiles, counted with the longest sequence, take more work items than a launch has (2^32): the
sequences go out in several launches.  Nearly all sequences are empty here; the same call without them gives the same results."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

pytestmark = pytest.mark.gpu

# sequences per launch at 65536 rows and one head: 10922 (dK/dV, d = 64), 16383, 32767 (forward, d = 64), 8191 (dK/dV, d = 192)
ROWS = {0: 3, 5: 130, 8190: 1, 8191: 33, 8192: 7, 10921: 64, 10922: 5, 16382: 2, 16383: 31, 16384: 70, 16390: 65536, 16398: 9}


@pytest.mark.parametrize("d,window", [(64, 0), (64, 70), (96, 0), (128, 70), (192, 0), (256, 70)])
def test_many_empty_sequences(d, window):
    import torch
    from paper_2605_15422_amd import binding as B, runner
    lens = np.zeros(16400, np.int64)
    lens[list(ROWS)] = list(ROWS.values())
    out = []
    for ls in (lens, lens[lens > 0]):
        print("case many", d, window, len(ls), flush=True)
        dg = B.upload(W.make_workload(W.Shape("many", len(ls), 40, 0, 0, 1, 1, d, window, seed=17), resp_lens=ls))
        b = runner.alloc(dg)
        runner.layer_step(dg, b)
        torch.cuda.synchronize()
        out.append({k: getattr(b, k).clone() for k in ("o_d", "lse_d", "dq_d", "dk_d", "dv_d", "dk_c2", "dv_c2")})
    for k, x in out[0].items():
        y = out[1][k]
        if k.endswith("c2"):   # (a prompt tile may be cut in another number of parts: one rounding of fp32 sums to bf16)
            assert (x.double() - y.double()).norm() <= 2.0**-8 * y.double().norm()
        else:
            assert not torch.isnan(x).any() and torch.equal(x.view(torch.int16), y.view(torch.int16))


@pytest.mark.parametrize("d", [64, 256])
def test_many_empty_groups(d):
    """Prompt tiles, too: every group gets as many as the longest prompt."""
    import torch
    import test_gpu_groups as G
    specs = [(40, [3, 70]), (65536, [33, 0, 5]), (1, []), (129, [64])]
    at = [7, 8190, 10922, 16399]   # where they stand among 16400 groups
    _, packed, table, cu = G._build(specs, 1, 1, d, 0, seed=23)
    many = np.zeros((16400, 4), np.int32)
    many[at] = table
    for g in range(len(many)):
        if g and g not in at:   # no prompt rows, no sequences
            many[g] = many[g - 1, 0] + many[g - 1, 1], 0, many[g - 1, 3], many[g - 1, 3]
    out = []
    for t in (many, table):
        print("case many groups", d, len(t), flush=True)
        out.append(G._run_groups([(65536, [])] * len(t), packed, t, cu, 1, 1, d, 0, 0)[1])
    for k, x in out[0].items():
        assert not torch.isnan(x).any() and torch.equal(x.view(torch.int16), out[1][k].view(torch.int16)), k
