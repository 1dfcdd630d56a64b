"""Rules that choose a route by the sizes of a call (csrc/rules.h), compiled for the host: the sizes of the GPU tests take the routes
that these tests are for, and choices that were measured to cost a tenth of a call."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++")

pytestmark = pytest.mark.skipif(CXX is None, reason="no host compiler")

SOURCE = r"""
#include <cstdio>
#include "rules.h"
using namespace dkv::rules;
int main() {
  int d, dq, n, longest, P, window, H, Hk, total;
  while (std::scanf("%d %d %d %d %d %d %d %d %d", &d, &dq, &n, &longest, &P, &window, &H, &Hk, &total) == 9) {
    const RowBlocks c{n, longest, P, window != 0, H / Hk, Hk, total};
    const int tile = d <= 128 ? 128 : d <= 256 ? 64 : 32;
    const long long prompt = (long long)((P + tile - 1) / tile) * Hk, resp = (long long)n * ((longest + tile - 1) / tile) * Hk;
    if (dq < 2) {
      const Waves w = choose_waves(c, d, dq, false);
      std::printf("%d %d\n", w.n, w.pair);
    } else {
      const Beside b = d <= 128 ? dq_beside(c, dq == 3, prompt, resp) : dq_beside_wide(c, dq == 3, d == 512, resp);
      std::printf("%d %d\n", prompt <= b.room ? b.waves : 0, prompt <= b.room && b.first);
    }
  }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("routes")
    (d / "routes.cpp").write_text(SOURCE)
    exe = str(d / "routes")
    subprocess.run([CXX, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2605_15422_amd", "csrc"), str(d / "routes.cpp"), "-o", exe],
                   check=True)

    def run(*args):
        r = subprocess.run([exe], input=" ".join(str(int(x)) for x in args), capture_output=True, text=True, check=True)
        return tuple(int(x) for x in r.stdout.split())
    return run


# (d, dQ, N, longest, P, window, H, H_k, rows), (waves, do workgroups share a CU)
WAVES = [
    ((128, 0, 8, 256, 517, 0, 32, 8, 1145), (4, True)),
    ((128, 0, 16, 1024, 8192, 0, 32, 8, 16384), (4, True)),
    ((128, 0, 16, 1992, 32768, 0, 32, 4, 25926), (8, False)),   # pairs 18.6 -> 19.1 ms
    ((128, 1, 16, 1992, 32768, 0, 32, 4, 25926), (4, True)),
    ((128, 0, 4, 100, 300, 0, 8, 2, 300), (4, False)),          # a CU each
    ((128, 0, 1, 3000, 0, 0, 16, 4, 3000), (4, False)),         # pairs 58 -> 60 us
    *(((d, 0, 70, 130, P, 0, 16, 4, 3570), (4, True)) for d in (64, 96, 128) for P in (1, 161)),   # test_gpu_half_tiles.py, edges
    ((128, 1, 70, 130, 161, 0, 16, 4, 3570), (4, True)),
    # the same: eight waves for one sequence, pairs for two
    *(((d, q, 1, P, 0, 0, H, Hk, P), (8, False) if d == 128 or not q else (8, True)) for d, H, Hk, P in
      ((96, 32, 8, 3393), (96, 8, 8, 13569), (128, 32, 8, 3393), (128, 8, 2, 16384)) for q in (0, 1)),
    *(((d, q, 2, P, 0, 0, H, Hk, 2 * P), (4, True)) for d, H, Hk, P in ((96, 32, 8, 3393), (128, 32, 8, 3393), (128, 8, 2, 16384)) for q in (0, 1)),
]


@pytest.mark.parametrize("case,waves", WAVES)
def test_waves(ask, case, waves):
    assert ask(*case) == waves


# (d, 2 or, several groups, 3, N, longest, P, window, H, H_k, rows), (waves of dQ in the launch, dQ first)
BESIDE = [
    # test_gpu_bwd_beside.py, one causal sequence
    *(((d, 2, 1, P, 0, 0, H, Hk, P), (w, 0)) for d in (64, 96, 128) for H, Hk, P, w in
      ((16, 4, 2081, 4), (8, 8, 2500, 4), (32, 8, 3873, 8), (8, 2, 16350, 8), (32, 8, 6657, 0))),
    *(((d, 2, 1, P, 0, 0, H, Hk, P), (w, 0)) for d, H, Hk, P, w in
      ((192, 2, 1, 65, 8), (192, 8, 2, 3001, 8), (192, 4, 4, 9600, 8), (256, 8, 2, 4097, 8), (256, 4, 4, 9700, 0), (512, 8, 2, 2049, 8), (512, 4, 2, 9700, 0))),
    # rows behind a prompt
    *(((d, 2, n, m, P, 0, H, Hk, T), (4, 1)) for d in (64, 96, 128) for H, Hk, P, n, m, T in
      ((32, 8, 4300, 2, 33, 53), (12, 4, 9000, 3, 130, 131), (8, 8, 4097, 7, 64, 448), (32, 4, 8321, 1, 97, 97))),
    *(((d, 2, n, m, P, 0, H, Hk, T), (8, f)) for d in (192, 256, 512) for H, Hk, P, n, m, T, f in
      ((8, 2, 3001, 3, 33, 53, 1), (12, 4, 70, 3, 700, 1381, 0))),
    ((64, 2, 17, 150, 31574, 0, 32, 8, 2300), (0, 0)),          # 2459 -> 2729 us
    ((128, 2, 1, 3000, 0, 512, 8, 8, 3000), (0, 0)),
    ((128, 3, 1, 3000, 0, 0, 8, 8, 3000), (0, 0)),              # several groups
    ((256, 3, 3, 33, 3001, 0, 8, 2, 53), (0, 0)),
    ((256, 2, 3, 33, 3001, 500, 8, 2, 53), (0, 0)),
]


@pytest.mark.parametrize("case,beside", BESIDE)
def test_beside(ask, case, beside):
    assert ask(*case) == beside
