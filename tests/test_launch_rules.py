"""Rules that size launches (csrc/rules.h), compiled for the host: what they choose where a wrong choice was measured to cost
a tenth of the call or more (MI355X), and what they may not choose."""
import os
import random
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
  long long v[14];
  char what;
  while (std::scanf(" %c", &what) == 1) {
    int n = 0;
    if (what == 'p' || what == 'k') {
      for (int i = 0; i < 13; ++i) std::scanf("%lld", &v[i]);
      if (what == 'k') std::scanf("%lld", &v[13]);
      PromptTiles c{v[0], (int)v[1], (int)v[2], (int)v[3], (int)v[4], (int)v[5], (int)v[6], (int)v[7], (int)v[8], v[9] != 0, v[10], (int)v[11]};
      if (what == 'k') c.head_dim = (int)v[13];
      n = what == 'k' ? pair_tiles(c, prompt_parts(c), prompt_parts(c, true)) : v[12] ? most_parts(c) : prompt_parts(c);
    }
    if (what == 'w') {
      for (int i = 0; i < 9; ++i) std::scanf("%lld", &v[i]);
      n = row_block_waves({(int)v[0], (int)v[1], (int)v[2], v[3] != 0, (int)v[4], (int)v[5]}, v[6] != 0, v[7] != 0, v[8] != 0);
    }
    if (what == 'r') {
      for (int i = 0; i < 3; ++i) std::scanf("%lld", &v[i]);
      n = replicate_copies(v[0], v[1], v[2]);
    }
    if (what == 'd') {
      std::scanf("%lld", &v[0]);
      n = dq_ring_slots((int)v[0]);
    }
    std::printf("%d\n", n);
  }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    exe = str(d / "rules")
    subprocess.run([CXX, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2605_15422_amd", "csrc"), str(d / "rules.cpp"), "-o", exe],
                   check=True)
    return lambda lines: [int(x) for x in subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True,
                                                         check=True).stdout.split()]


def _parts(d, N, P, total, longest, H, Hk, shared=-1, groups=1, most=0):
    tile = 128 if d <= 128 else 64 if d <= 256 else 32
    tiles = groups * -(-P // tile) * Hk
    return "p " + " ".join(str(int(x)) for x in (tiles, N, groups, total, longest, H // Hk, Hk, tile, 16 if d == 512 else 32,
                                                  d == 512, shared, P, most))


# (d, N, P, total, longest, H, H_k, shared), the counts within a tenth of the best one
PARTS = [
    ((64, 19, 34, 120, 7, 8, 2), range(10, 33)),        # one row block a sequence: 1 part 61 us, 19 parts 22
    ((512, 16, 21, 96, 7, 12, 4), range(8, 17)),        # 1 part 38 us, 16 parts 25
    ((128, 23, 132, 1075, 60, 8, 8), (2, 3, 4, 5, 6)),  # 23 parts 53 us, 4 parts 32
    ((64, 6, 3043, 204, 60, 8, 8), (1,)),               # 3 parts 98 us, 1 part 76
    ((128, 7, 793, 475, 100, 16, 16), (1, 2)),          # 5 parts 106 us, 1 part 65
    ((128, 10, 1259, 68, 8, 8, 8, 96), (1,)),          # with 2 parts dK/dV and dQ do not share a launch: 42 -> 64 us
    ((128, 15, 67, 97, 7, 32, 8, 16), range(8, 33)),    # dQ's walk is short: 2 parts 55 us, 15 parts 40
    ((128, 2, 1607, 2129, 1500, 32, 4), (1, 2)),        # 4 parts 434 us, 2 parts 378
]


@pytest.mark.parametrize("case,good", PARTS)
def test_prompt_parts(ask, case, good):
    assert ask([_parts(*case)])[0] in good


def test_prompt_parts_keep_sums_that_have_one_result(ask):
    """Two adds to zero commute, three do not: calls for which 512 workgroups mean at most two parts get at most two."""
    rng = random.Random(5)
    few = more = 0
    lines = []
    for _ in range(4000):
        N, R = rng.randint(1, 40), rng.randint(1, 3000)
        Hk = rng.choice([1, 2, 4, 8, 16])
        args = (rng.choice([64, 96, 128, 192, 256, 512]), N, rng.randint(1, 20000), N * R, R, Hk * rng.choice([1, 3, 4, 8]), Hk,
                rng.randint(-1, 600), rng.choice([1, 1, min(N, 3)]))
        lines += [_parts(*args, most=1), _parts(*args)]
    got = ask(lines)
    for most, n in zip(got[::2], got[1::2]):
        assert 1 <= n <= 32
        if most <= 2:
            assert n <= most
            few += 1
        else:
            more += n > 2
    assert few > 500 and more > 500


# (d, N, P, total, longest, H, H_k, shared), two dK/dV workgroups a CU?
PAIRS = [
    ((128, 16, 8192, 16384, 1024, 32, 8), 1),       # 4.12 -> 3.70 ms
    ((96, 8, 4111, 7300, 1680, 16, 4), 1),          # 699 -> 590 us
    ((96, 5, 11889, 132, 31, 32, 8), 1),            # 136 -> 108
    ((128, 1, 3577, 3577, 3577, 12, 4), 0),         # 271 -> 364
    ((128, 7, 71, 13933, 2878, 8, 8), 0),           # responses: 263 -> 316
    ((128, 4, 2567, 4300, 1829, 4, 2), 0),          # 116 -> 140
    ((96, 7, 4639, 581, 118, 4, 2), 0),             # 44 -> 48
    ((128, 1, 3999, 101, 101, 4, 2), 0),            # 64 workgroups: 22 -> 23
    ((128, 16, 8192, 16384, 1024, 32, 8, 4000), 0),  # dQ shares the launch
    ((128, 6, 9832, 13032, 2474, 32, 4), 0),        # 4.44 -> 4.70 ms
    # two and a quarter to two and three quarters rounds of 256 are as many of 512: three of the one against one full and one half
    # of the other, which at d = 128 is slower
    ((128, 16, 9216, 16384, 1024, 32, 8), 0),       # 5.70 -> 5.78 ms
    ((128, 16, 10240, 16384, 1024, 32, 4), 0),      # 5.65 -> 5.75
    ((128, 9, 19149, 18400, 2443, 12, 4), 0),       # 4.99 -> 5.07
    ((128, 8, 17500, 16384, 2048, 16, 4), 0),       # 5.60 -> 5.69
    ((96, 16, 8660, 6500, 489, 32, 8), 1),          # 1.90 -> 1.80
    ((128, 8, 3072, 8192, 1024, 8, 2), 0),          # 308 -> 331 us in nine parts
    ((128, 4, 0, 4000, 1000, 32, 8), 0),
    ((128, 4, 8192, 0, 0, 32, 8), 0),
    # the sizes of test_gpu_dkdv_pair.py
    ((128, 8, 1537, 655, 300, 64, 32), 1),
    ((96, 8, 1537, 655, 300, 64, 32), 1),
    ((128, 6, 4097, 1199, 515, 8, 4), 1),
    ((96, 6, 4097, 1199, 515, 8, 4), 1),
    *(((d, N, P, total, longest, H, Hk), 1) for d in (96, 128)
      for N, P, total, longest, H, Hk in ((4, 4097, 534, 301, 8, 8), (4, 9001, 262, 129, 12, 4), (4, 4097, 534, 301, 32, 8), (3, 8100, 198, 100, 32, 4))),
]


@pytest.mark.parametrize("case,pair", PAIRS)
def test_pair_tiles(ask, case, pair):
    line = _parts(*case)
    assert ask(["k" + line[1:] + " %d" % case[0]]) == [pair]


@pytest.mark.parametrize("d,per_cu", [(64, 3), (96, 2), (128, 1)])
def test_dq_rings_fit_the_lds(ask, d, per_cu):
    """As many workgroups as their registers let on a CU (test_kernel_registers.py): 160 KB for K and V tiles of 64 keys."""
    slots, = ask(["d %d" % d])
    assert slots >= 3 and per_cu * slots * 2 * 64 * 2 * d <= 160 * 1024


# (d, dQ, N, longest, P, window, H, H_k), waves, what they save
WAVES = [
    ((128, 0, 1, 1021, 0, 0, 32, 8), 4),         # forward 35 -> 25 us
    ((128, 0, 22, 135, 392, 0, 8, 8), 8),        # four: 25 -> 32 us
    ((128, 1, 22, 135, 392, 0, 8, 8), 8),        # four: 26 -> 38
    ((128, 0, 22, 127, 392, 0, 8, 8), 4),        # 23 -> 18: every sequence is one row block of four waves
    ((128, 0, 24, 119, 5407, 0, 16, 16), 4),     # 309 -> 195: and one of eight, half of them without rows
    ((128, 0, 18, 253, 139, 0, 8, 1), 8),        # four: 19 -> 27
    ((128, 1, 18, 253, 139, 0, 8, 1), 8),        # four: 23 -> 32
    ((128, 0, 1, 1229, 0, 918, 32, 4), 8),       # four: 39 -> 56
    ((128, 0, 1, 1475, 0, 0, 32, 8), 4),         # 42 -> 31, more than a workgroup a CU
    ((128, 0, 1, 10746, 0, 0, 4, 2), 4),         # 248 -> 185
    ((128, 0, 2, 3478, 753, 0, 8, 8), 4),        # 124 -> 98
    ((128, 0, 1, 10723, 0, 0, 8, 8), 8),         # four: 288 -> 304
    ((128, 1, 23, 496, 4793, 0, 4, 2), 8),       # four: 176 -> 243
    ((128, 1, 20, 26, 4283, 0, 8, 8), 8),        # four: 88 -> 92
    ((64, 0, 37, 296, 10, 0, 32, 4), 4),         # eight: 40 -> 47
    ((64, 0, 31, 314, 2722, 0, 16, 4), 4),       # eight: 156 -> 178
    ((64, 1, 39, 1040, 500, 0, 32, 8), 4),       # eight: 588 -> 775
    ((96, 0, 34, 12, 2797, 0, 32, 4), 8),        # four: 74 -> 102
    ((96, 1, 34, 40, 2797, 0, 32, 4), 4),
    ((128, 0, 16, 1024, 8192, 0, 32, 8), 8),
]


@pytest.mark.parametrize("case,waves", WAVES)
def test_row_block_waves(ask, case, waves):
    d, dq, N, longest, P, window, H, Hk = case
    pair = d == 64 or (d == 96 and dq)
    assert ask(["w " + " ".join(map(str, (N, longest, P, window, H // Hk, Hk, int(pair), dq, 0)))]) == [waves]


def test_a_shared_launch_takes_four_waves(ask):
    assert ask(["w 20 26 0 0 1 8 0 1 1", "w 1 1 0 0 1 1 0 1 1"]) == [4, 4]


# (N, P, T), copies of a prompt row per workgroup of the replicating copy
@pytest.mark.parametrize("case,copies", [((16, 8192, 16384), 16), ((23, 29, 138), 2), ((16, 64, 264), 4), ((4, 32, 27), 1),
                                         ((1, 100000, 0), 16), ((0, 0, 0), 1), ((2**31 - 1, 2**31 - 1, 0), 16)])
def test_replicate_copies(ask, case, copies):
    assert ask(["r %d %d %d" % case]) == [copies]
