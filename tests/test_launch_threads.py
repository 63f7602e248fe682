"""CPU check: no forward launch asks for 2^32 threads or more.

A dispatch counts its threads in 32 bits, and a larger grid is cut without an error: part
of the field would not be written.  Volumes a few voxels wide reach that with short
z-chunks, at most 64 voxels of a wave's 64 lanes being used; the volumes here are among the
narrowest and the largest that the entry points take and a device of 288 GB holds."""
import ctypes
import os
import random

import pytest

from conftest import ROOT

LIB = os.path.join(ROOT, "paper_2004_05962_amd", "libbsi_check.so")

CASES = [
    ((1, 65536, 26500), (4, 4, 4)),     # 1.7e9 rows of one voxel: 21 GB
    ((1, 44721, 44721), (5, 5, 5)),     # the most rows
    ((11, 1907, 1 << 20), (1, 1, 1)),
    ((12, 1 << 20, 1907), (3, 3, 3)),
    ((65, 33000, 33000), (16, 16, 16)),
    ((65, 1 << 20, 350), (64, 64, 64)),
    ((2000, 3400, 3500), (5, 5, 5)),
]
RNG = random.Random(11)
for _ in range(200):
    nx = int(2 ** RNG.uniform(0, 12))
    rows = min(1.9e9, 288e9 / (12 * nx))
    ny = int(min(1 << 20, max(rows / (1 << 20) + 1, 2 ** RNG.uniform(0, 20))))
    nz = int(min(1 << 20, rows / ny))
    CASES.append(((nx, ny, nz), tuple(RNG.choice([1, 2, 3, 4, 5, 7, 8, 16, 40, 64]) for _ in range(3))))


def test_forward_launches_stay_below_2_to_the_32_threads():
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} is not built: run __graft_entry__.build()")
    L = ctypes.CDLL(LIB)
    i3 = ctypes.c_int32 * 3
    out = (ctypes.c_int64 * 4)()
    for dims, spacing in CASES:
        rc = L.bsi_check_launch_threads(i3(*dims), i3(*spacing), out)
        if rc == -1:
            continue  # a plane of more voxels than the entry points take
        assert rc == 0, (dims, spacing)
        assert max(out) < 1 << 32, (dims, spacing, list(out))
