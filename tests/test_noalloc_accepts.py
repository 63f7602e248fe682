"""CPU: every geometry within bsi_adjoint_noalloc's limit is taken, whatever bricks the
kernels use: its partials fit the fixed scratch.

The limit is the size of the partials in bricks of 64 x 16 voxel columns (limit_bytes).
Narrow widths at x spacings 1 and 2 and a last z-tile of its own once did not fit."""
import ctypes
import random

import pytest

from conftest import has_gpu
from paper_2004_05962_amd import _lib
from test_noalloc_limit import CAP, limit_bytes

pytestmark = pytest.mark.skipif(has_gpu(), reason="needs the no-device path")

SIZES = [
    ((991, 885, 107), (1, 20, 12)),     # 9 z-tiles, the last one short
    ((55, 7000, 32), (1, 10, 1)),
    ((61, 7657, 33), (1, 20, 1)),
    ((34, 6200, 33), (2, 1, 1)),
    ((42, 8002, 20), (2, 1, 1)),
    ((62, 2175, 30), (1, 1, 1)),
]


def taken(dims, spacing):
    # the call ends where it finds no device (the pointers are not followed)
    rc = _lib.lib().bsi_adjoint_noalloc(ctypes.c_void_p(256), _lib._triple(dims, "dims"),
                                        _lib._triple(spacing, "spacing"), ctypes.c_void_p(256), ctypes.c_void_p(0))
    assert rc in (_lib.BSI_ERR_NO_DEVICE, _lib.BSI_ERR_UNSUPPORTED)
    return rc == _lib.BSI_ERR_NO_DEVICE


@pytest.mark.parametrize("dims,spacing", SIZES)
def test_sizes_near_the_limit(dims, spacing):
    assert limit_bytes(dims, spacing) <= CAP
    assert taken(dims, spacing)


@pytest.mark.parametrize("dx", [1, 2, 3, 5, 16])
def test_every_narrow_width(dx):
    """For every width, the longest volume that the limit takes."""
    rng = random.Random(dx)
    for nx in range(1, 200):
        sy, sz = rng.choice([1, 1, 2, 7, 20, 64]), rng.choice([1, 1, 2, 3, 12])
        ny = rng.randint(1, 3000)
        lo, hi = 0, 1 << 20
        while lo < hi:  # (the limit is not quite monotone in nz: any size near it will do)
            mid = (lo + hi + 1) // 2
            if limit_bytes((nx, ny, mid), (dx, sy, sz)) <= CAP:
                lo = mid
            else:
                hi = mid - 1
        if lo == 0 or ny * lo > 1.9e9:
            continue
        for nz in (lo, max(1, lo - 1), max(1, lo - sz)):
            dims, spacing = (nx, ny, nz), (dx, sy, sz)
            assert taken(dims, spacing) == (limit_bytes(dims, spacing) <= CAP), (dims, spacing)
