"""CPU check of the real-spacing adjoint's table reads in bricks with empty cells.

With two-plane slabs a cell past the volume marches all the same, for the barriers:
what it reads of the per-axis tables must lie inside them too."""
import ctypes
import os

import pytest

from conftest import ROOT

LIB = os.path.join(ROOT, "paper_2004_05962_amd", "libbsi_check.so")


@pytest.mark.parametrize("dims", [(26, 7, 2000), (26, 23, 2000), (3000, 18, 60), (3001, 7, 61), (27, 17, 31), (1, 1, 40)])
@pytest.mark.parametrize("spacing,origin", [((1.0, 1.0, 1.0), (0.0, 0.0, 0.0)), ((1.25, 1.0, 1.5), (-1.0, 0.0, -0.5)),
                                            ((3.5, 1.2, 1.0), (-3.0, -0.7, 0.0))])
def test_cell_weights_are_read_inside_the_tables(dims, spacing, origin):
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} is not built: run __graft_entry__.build()")
    L = ctypes.CDLL(LIB)
    f3 = ctypes.c_float * 3
    msg = ctypes.create_string_buffer(512)
    rc = L.bsi_check_general_indices((ctypes.c_int32 * 3)(*dims), f3(*spacing), f3(*origin), msg, 512)
    assert rc == 0, msg.value.decode()
