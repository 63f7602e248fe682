"""CPU check of the fused SSD step's order of LDS accesses.

The order of a workgroup's loads, stores and barriers is one routine, which the kernel
and this check both run (fused_start, fused_walk).  Here each access is recorded with
the barrier interval it falls in: a region that one wave stores and another reads or stores again
must have a barrier between the two, and every read must find the plane it is
meant for.  Waves of a workgroup meet at barriers only, so an order that holds here
holds for any speed of the waves."""
import ctypes
import os

import pytest

from conftest import ROOT

LIB = os.path.join(ROOT, "paper_2004_05962_amd", "libbsi_check.so")

# dims, spacing, z-bricks per workgroup, slabs of every plane (None: as it comes)
CASES = [
    ((64, 64, 40), (5, 5, 5), 1, 1),
    ((256, 256, 160), (5, 5, 5), 1, 1),
    ((512, 300, 199), (5, 5, 5), 1, 1),       # a partial last tile
    ((512, 510, 199), (5, 5, 5), 4, 1),       # every z-brick in one workgroup
    ((1024, 260, 210), (5, 5, 5), 1, 1),
    ((200, 220, 240), (2, 3, 1), 5, 0),       # several z-bricks per workgroup
    ((300, 260, 40), (5, 5, 1), 2, 1),        # a z-tile per plane
    ((64, 64, 200), (1, 1, 1), 1, 0),
    ((300, 256, 200), (1, 1, 1), 2, 0),       # two-plane slabs, several z-bricks
    ((40, 70, 21), (12, 35, 7), None, 1),
    ((5, 5, 1), (1, 1, 1), 1, 0),             # one plane
    ((1, 40, 50), (3, 3, 3), None, 1),
    ((70, 33, 129), (2, 3, 64), None, 0),
    ((30, 33, 129), (2, 3, 64), None, 0),     # narrow bricks: two-plane slabs
]


@pytest.mark.parametrize("dims,spacing,deep,whole", CASES)
def test_lds_accesses_are_ordered_by_barriers(dims, spacing, deep, whole):
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} is not built: run __graft_entry__.build()")
    L = ctypes.CDLL(LIB)
    i3 = ctypes.c_int32 * 3
    info = (ctypes.c_int32 * 2)()
    msg = ctypes.create_string_buffer(512)
    rc = L.bsi_check_fused(i3(*dims), i3(*spacing), info, msg, 512)
    assert rc == 0, msg.value.decode()
    if deep is not None:
        assert info[0] == deep
    if whole is not None:
        assert info[1] == whole
