"""The head-dim 64 / 96 / 128 forward and dQ kernels run four or eight waves in a workgroup, chosen by the number of row
blocks: both counts at row counts around the 32-row subtiles and the 64-key tiles, with and without a window."""
import numpy as np
import pytest

from paper_2605_15422_amd import workloads as W

import parity_util as PU

pytestmark = pytest.mark.gpu

FEW = [33, 64, 1, 0, 97]                                            # a handful of workgroups: four waves
MANY = [(13 * i) % 71 for i in range(200)] + [31, 32, 33, 63, 64, 65, 129]   # more than the 256 CUs: eight


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("lens", [FEW, MANY], ids=["few", "many"])
@pytest.mark.parametrize("window", [0, 45])
def test_wave_counts(d, lens, window):
    print("case waves", d, len(lens), window, flush=True)
    shape = W.Shape("waves", len(lens), 67, 0, 0, 8, 2, d, window, seed=50 + d + len(lens))
    PU.bounded_parity(W.make_workload(shape, resp_lens=np.asarray(lens)))
