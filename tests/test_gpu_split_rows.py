"""GPU parity of the kernels for head dims 96 and 192, whose 192- and 384-byte rows do not divide the 1 KB of a load
instruction and whose dK/dV (at 192 also forward and dQ) kernels have a wave of its own for the requests.  Sizes around the
32-, 64- and 128-key tiles, the 32-row blocks and the LDS stages; bounds as in parity_util."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

import parity_util as PU

pytestmark = pytest.mark.gpu

CASES = [
    # name, N, P, lens, H, Hk, window
    ("rows", 6, 67, [15, 16, 17, 31, 33, 129], 4, 2, 0),
    ("g1", 2, 129, [70, 140], 2, 2, 0),
    ("g3", 2, 128, [64, 96], 6, 2, 0),
    ("g8", 2, 191, [64, 100], 8, 1, 0),
    ("long", 2, 700, [300, 45], 4, 1, 0),
    ("win_tile", 3, 200, [150, 64, 33], 4, 2, 64),
    ("win_odd", 2, 130, [260, 90], 2, 1, 97),
    ("win_one_key", 2, 70, [40, 1], 2, 1, 1),
    ("p0", 2, 0, [130, 31], 4, 2, 0),
    ("empty", 3, 48, [0, 20, 0], 4, 2, 0),
    ("all_empty", 2, 40, [0, 0], 2, 1, 0),
    ("one_block", 1, 33, [21], 1, 1, 0),
    ("win_one_block", 1, 70, [30], 1, 1, 8),
    ("seven_blocks", 1, 3, [224], 1, 1, 0),
]


@pytest.mark.parametrize("d", [96, 192])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_parity(case, d):
    from paper_2605_15422_amd import binding as B
    name, N, P, lens, H, Hk, win = case
    print("case", name, d, flush=True)
    shape = W.Shape("%s_d%d" % (name, d), N, P, 0, 0, H, Hk, d, win, seed=909 + len(name))
    PU.full_parity(W.make_workload(shape, resp_lens=np.asarray(lens)), flags=B.FLAG_ACCUM_CTX_F32 if name in ("g3", "long") else 0)
