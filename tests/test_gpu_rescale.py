"""Forward at head dims 64 to 128 where the scores jump by more than the fp32 exponent range inside a tile: the reference of the
exponentials is then moved after the probabilities have overflowed, with four and with eight waves, with and without a window."""
import numpy as np
import pytest

import parity_util as PU
from oracle import attention_oracle as orc
from paper_2605_15422_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("N,window", [(3, 0), (3, 45), (20, 0)])
def test_jumping_scores(d, N, window):
    print("case jumping scores", d, N, window, flush=True)
    lens = np.asarray([200] + [10] * (N - 1))
    wl = W.make_workload(W.Shape("jump", N, 100, 0, 0, 8, 8, d, window, seed=4100 + d), resp_lens=lens)

    def scaled(bits, factor):
        return W.f32_to_bf16_bits((W.bf16_bits_to_f32(bits) * factor).astype(np.float32))

    big_c, big_d = np.full(100, 0.125, np.float32), np.full(int(lens.sum()), 0.125, np.float32)
    big_c[[3, 37, 70]] = [2.0, 6.0, 16.0]      # both halves of a 64-key tile, then the next tile
    big_d[[0, 33, 101, 190]] = [8.0, 16.0, 24.0, 32.0]
    wl.q_c, wl.q_d = scaled(wl.q_c, 16.0), scaled(wl.q_d, 16.0)
    wl.k_c, wl.k_d = scaled(wl.k_c, big_c[:, None, None]), scaled(wl.k_d, big_d[:, None, None])
    x = PU.oracle_inputs(wl)
    ref = orc.dualkv_forward(x["q_c"], x["k_c"], x["v_c"], x["q_d"], x["k_d"], x["v_d"], wl.cu_seqlens, wl.scale, window)
    dg, b = PU.run_hip_layer(wl)
    rep = []
    for part, o, lse in (("c", b.o_c, b.lse_c), ("d", b.o_d, b.lse_d)):
        PU.compare("O_" + part, PU.to_f64(o), ref["o_" + part], rep)
        # |LSE| reaches hundreds: the fp32 sum of d products behind it carries a few 2^-24 of that
        want = ref["lse_" + part]
        err = np.abs(PU.to_f64(lse) - want)
        assert (err <= PU.LSE_TOL + 2.0 ** -20 * np.abs(want)).all(), err.max()
    print("\n".join(rep), flush=True)
