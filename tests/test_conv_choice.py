"""The convolution's automatic choice of a kernel (host only, no GPU): layers on
which the channel-block kernels were measured slower than the general ones go to
the general ones, layers that gain from them stay, and every choice is one that
the library can launch.  The times behind each line are microseconds, general
kernel against channel blocks, on 256 CUs."""
from __future__ import annotations

import random

import pytest

import paper_2005_06410_amd as lt
from synth import conv as sc

STAGED, DIRECT, BLOCKS, RUNS = 1, 2, 3, 4

# kn, k, ci, hi, wi, b, stride, pad
GENERAL = [
    (16, 1, 16, 112, 112, 10, 1, 0),     # 7.5 against 35.0: one group, sixteen waves to a tile
    (4, 1, 64, 112, 112, 10, 1, 0),      # 14.5, 39.4
    (16, 1, 128, 112, 112, 10, 1, 0),    # 24.4, 40.8
    (32, 1, 32, 112, 112, 10, 1, 0),     # 11.6, 17.2
    (64, 1, 16, 112, 112, 10, 1, 0),     # 10.6, 17.5
    (4, 3, 16, 112, 112, 10, 1, 0),      # 24.3, 36.6
    (33, 1, 64, 112, 112, 10, 1, 0),     # 20.0, 35.5: filters loaded one by one
    (33, 3, 16, 112, 112, 10, 1, 1),     # 40.6, 49.2
    (11, 1, 12, 88, 125, 61, 3, 0),      # 7.5, 23.5
    (111, 1, 128, 93, 83, 3, 1, 0),      # 15.1, 20.6
    (298, 2, 40, 132, 52, 10, 4, 0),     # 14.3, 19.2: partial blocks
    (376, 7, 24, 29, 178, 5, 1, 0),      # 170, 221
    (603, 5, 31, 53, 17, 20, 1, 0),      # 122, 158
]
KEPT = [
    (384, 3, 384, 13, 13, 1, 1, 0),      # 61.8, 15.9: AlexNet's seventh layer on one image
    (384, 3, 192, 27, 27, 16, 1, 1),     # 270, 134
    (192, 5, 64, 55, 55, 80, 1, 0),      # 1022, 924
    (33, 3, 64, 28, 28, 7, 1, 1),
    (16, 3, 128, 28, 28, 7, 1, 0),
    (2, 5, 33, 31, 12, 28, 1, 1),        # 39.3, 9.0
]


def choice(c):
    kn, k, ci, hi, wi, b, s, p = c
    return lt.conv_choice(kn, k, k, ci, hi, wi, b, s, p)


@pytest.mark.parametrize("case", GENERAL)
def test_layers_that_channel_blocks_slow_down_go_to_the_general_kernels(case):
    unit = case[6] == 1 and case[7] == 0
    assert choice(case)[0] == (DIRECT if unit else STAGED)


@pytest.mark.parametrize("case", KEPT)
def test_layers_that_gain_from_channel_blocks_keep_them(case):
    assert choice(case)[0] == BLOCKS


# kn, k, ci, hi, wi, b, stride; the LDS-staged 128 x 128 tile against runs of taps
@pytest.mark.parametrize("case,family", [
    ((384, 9, 3, 158, 192, 42, 3), STAGED),      # 258 against 316
    ((640, 6, 8, 223, 155, 25, 3), STAGED),      # 371, 446
    ((256, 10, 8, 114, 150, 26, 2), STAGED),     # 381, 423
    ((384, 8, 3, 158, 192, 42, 3), RUNS),
    ((640, 7, 8, 223, 155, 25, 3), RUNS),
    ((256, 11, 8, 114, 150, 26, 2), RUNS),
    ((96, 9, 3, 158, 192, 42, 3), RUNS),         # no 128 x 128 tile
    ((384, 9, 3, 58, 92, 4, 3), RUNS),           # too few of them
])
def test_wasteful_runs_go_to_the_wide_staged_tile(case, family):
    kn, k, ci, hi, wi, b, s = case
    assert lt.conv_choice(kn, k, k, ci, hi, wi, b, s, 0)[0] == family


def test_every_choice_can_be_launched():
    legal = {(STAGED, 64, 64, 1), (STAGED, 128, 128, 1),
             (DIRECT, 64, 64, 1), (DIRECT, 64, 64, 2), (DIRECT, 64, 64, 4), (DIRECT, 64, 128, 1), (DIRECT, 128, 64, 1),
             (BLOCKS, 64, 128, 1), (BLOCKS, 64, 32, 4), (BLOCKS, 64, 32, 8), (BLOCKS, 64, 16, 4), (BLOCKS, 64, 16, 8),
             (BLOCKS, 32, 32, 8), (BLOCKS, 32, 64, 8), (BLOCKS, 16, 16, 16), (RUNS, 64, 32, 2), (RUNS, 64, 32, 4)}
    rng = random.Random(3)
    seen = set()
    for _ in range(20000):
        k = rng.choice([1, 2, 3, 4, 5, 6, 7, 9, 11, 40])
        s, p = rng.choice([1, 1, 2, 3, 4]), rng.choice([0, 0, k // 2, k])
        kn, ci = rng.choice([rng.randint(1, 40), 128 * rng.randint(1, 6), rng.randint(1, 700)]), rng.randint(1, 600)
        hi, wi, b = rng.randint(k, 300), rng.randint(k, 300), rng.randint(1, 64)
        if hi * wi * ci * b >= 1 << 30:
            continue
        c = lt.conv_choice(kn, k, k, ci, hi, wi, b, s, p)
        assert c in legal, (kn, k, ci, hi, wi, b, s, p)
        assert not (c[0] == DIRECT and (p or s > 1 or k * k * ci > 16384))
        assert not (c[0] == RUNS and (p or s == 1 or kn % 4 or k < 4))
        seen.add(c)
    assert {c[0] for c in seen} == {STAGED, DIRECT, BLOCKS, RUNS}


def test_choice_checks_its_arguments():
    assert lt.conv_choice(4, 3, 3, 8, 9, 9, 0) == (0, 0, 0, 0)       # an empty batch launches nothing
    lib = lt.load()
    assert lib.convgemm_choice(0, 3, 3, 8, 9, 9, 1, 1, 0, None) == -1
    assert lib.convgemm_choice(4, 3, 3, 8, 2, 9, 1, 1, 0, None) == -5
    assert lib.convgemm_choice(4, 3, 3, 8, 9, 9, 1, 1, 0, None) == -10


@pytest.mark.parametrize("spec", sc.ALEXNET_CONV, ids=lambda s: f"layer{s['layer']}")
@pytest.mark.parametrize("b", [1, 80])
def test_alexnet_layers_run_on_the_strided_and_channel_block_kernels(spec, b):
    c = lt.conv_choice(spec["kn"], spec["kh"], spec["kw"], spec["ci"], spec["hi"], spec["wi"], b, spec["s"], spec["p"])
    assert c[0] == (RUNS if spec["ci"] == 3 else BLOCKS)
