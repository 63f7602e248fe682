"""CPU check of the fused SSD step's LDS layout, staging map and reads of the finished
planes, over every spacing and ragged volumes (tests/test_fused_order.py has the order of
its accesses)."""
import ctypes
import os
import random

import pytest

from conftest import ROOT

LIB = os.path.join(ROOT, "paper_2004_05962_amd", "libbsi_check.so")


def check(dims, spacing):
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} is not built: run __graft_entry__.build()")
    L = ctypes.CDLL(LIB)
    i3 = ctypes.c_int32 * 3
    msg = ctypes.create_string_buffer(512)
    rc = L.bsi_check_fused(i3(*dims), i3(*spacing), (ctypes.c_int32 * 2)(), msg, 512)
    assert rc == 0, (dims, spacing, msg.value.decode())


@pytest.mark.parametrize("d", range(1, 65))
def test_every_spacing(d):
    check((3 * d + 55, 2 * d + 37, d + 9), (d, max(1, d // 2), min(64, d + 3)))


def test_random_geometries():
    rng = random.Random(3)
    for _ in range(300):
        spacing = [rng.choice([1, 1, 2, 2, 3, 4, 5, 7, 11, 30, 64]) for _ in range(3)]
        check([max(1, int(2 ** rng.uniform(0, 9))) for _ in range(3)], spacing)
