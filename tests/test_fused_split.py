"""CPU check of how the fused SSD step cuts a volume into workgroups.

One workgroup runs per CU (two where bricks are narrow), so the launch takes rounds of 256
(512) workgroups, and a round costs a workgroup's planes and about 9 planes more.  A
launch a little above a whole round leaves almost a whole round idle: the split
taken must cost no more than any other, by that count."""
import ctypes
import os
import random

import pytest

from conftest import ROOT

LIB = os.path.join(ROOT, "paper_2004_05962_amd", "libbsi_check.so")
START = 9

SIZES = [
    ((512, 400, 220), (6, 6, 6)),
    ((152, 343, 409), (3, 3, 3)),
    ((532, 230, 81), (6, 2, 8)),
    ((200, 220, 240), (2, 3, 1)),
    ((256, 256, 160), (5, 5, 5)),
    ((64, 64, 40), (5, 5, 5)),
    ((2, 4096, 2000), (5, 5, 5)),
    ((1, 1, 1), (1, 1, 1)),
    ((1500, 1400, 300), (4, 4, 4)),
    ((300, 256, 200), (1, 1, 1)),
]


def test_no_other_split_is_cheaper():
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} is not built: run __graft_entry__.build()")
    L = ctypes.CDLL(LIB)
    i3 = ctypes.c_int32 * 3
    rng = random.Random(7)
    sizes = SIZES + [([int(2 ** rng.uniform(4, 9.5)) for _ in range(3)], [rng.choice([1, 2, 3, 4, 5, 6, 8, 12, 20])] * 3)
                     for _ in range(200)]
    for dims, spacing in sizes:
        out = (ctypes.c_int32 * 6)()
        assert L.bsi_check_fused_split(i3(*dims), i3(*spacing), out) == 0
        columns, bricks, planes, deep, nz, chip = out
        assert chip in (256, 512)
        assert nz == -(-bricks // deep)

        def cost(k):
            return -(-columns * -(-bricks // k) // chip) * (min(k * planes, dims[2]) + START)
        # (splits into more than 16 rounds are left out: a round is then small)
        best = min(cost(k) for k in range(1, bricks + 1) if k == bricks or columns * -(-bricks // k) <= 16 * chip)
        assert cost(deep) <= best, (dims, spacing, list(out), best)
