"""The head-dim 64 / 96 / 128 forward and dQ kernels run four or eight waves in a workgroup, chosen by the number of row
blocks: row counts around the 32-row subtiles and the 64-key tiles, with and without a window, and enough rows of one
length, head dim 64, to keep every CU busy several times over."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

import parity_util as PU

pytestmark = pytest.mark.gpu

FEW = [33, 64, 1, 0, 97]                                            # a handful of workgroups: four waves
# 1, 2, 3, 4 and 8 heads a KV head, packed into four waves or, three, each by itself
LONG = [(1, 1, [4000, 4000]), (2, 1, [3200, 3100, 33]), (3, 1, [2200, 2100]), (4, 1, [1600] * 3), (8, 1, [800] * 3 + [31])]
MANY = [(13 * i) % 71 for i in range(200)] + [31, 32, 33, 63, 64, 65, 129]   # more than the 256 CUs: eight


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("lens", [FEW, MANY], ids=["few", "many"])
@pytest.mark.parametrize("window", [0, 45])
def test_wave_counts(d, lens, window):
    print("case waves", d, len(lens), window, flush=True)
    shape = W.Shape("waves", len(lens), 67, 0, 0, 8, 2, d, window, seed=50 + d + len(lens))
    PU.bounded_parity(W.make_workload(shape, resp_lens=np.asarray(lens)))


@pytest.mark.parametrize("H,Hk,lens", LONG, ids=["g%d" % x[0] for x in LONG])
@pytest.mark.parametrize("window", [0, 100])
def test_twelve_waves(H, Hk, lens, window):
    """Sampled rows against the oracle's one-row evaluation (the dense oracle would need minutes at these sizes)."""
    import torch
    from paper_2605_15422_amd import binding as B, runner
    print("case twelve", H, lens, window, flush=True)
    wl = W.make_workload(W.Shape("twelve", len(lens), 200, 0, 0, 24 * H, 24 * Hk, 64, window, seed=70 + H), resp_lens=np.asarray(lens))
    dg = B.upload(wl)
    b = runner.alloc(dg)
    runner.layer_step(dg, b)
    torch.cuda.synchronize()
    f = W.bf16_bits_to_f64
    rng = np.random.default_rng(H)
    for _ in range(24):
        i = int(rng.integers(len(lens)))
        r = int(rng.choice([0, 1, 31, 32, 63, lens[i] - 1, int(rng.integers(lens[i]))]))
        r = min(r, lens[i] - 1)
        h = int(rng.integers(24 * H))
        r0, hk = int(wl.cu_seqlens[i]), h // H
        k = np.concatenate([f(wl.k_c[:, hk]), f(wl.k_d[r0:r0 + r + 1, hk])])
        v = np.concatenate([f(wl.v_c[:, hk]), f(wl.v_d[r0:r0 + r + 1, hk])])
        q, do = f(wl.q_d[r0 + r, h]), f(wl.do_d[r0 + r, h])
        lo = max(0, 200 + r - window + 1) if window else 0
        s = (k[lo:] @ q) * wl.scale
        lse = s.max() + np.log(np.exp(s - s.max()).sum())
        p = np.exp(s - lse)
        o = p @ v[lo:]
        dq = wl.scale * (p * (v[lo:] @ do - o @ do)) @ k[lo:]
        rep = []
        PU.compare("O", PU.to_f64(b.o_d[r0 + r, h]), o, rep)
        PU.compare_lse("LSE", PU.to_f64(b.lse_d[h, r0 + r:r0 + r + 1]), np.asarray([lse]), rep)
        PU.compare("dQ", PU.to_f64(b.dq_d[r0 + r, h]), dq, rep)
