"""CPU: where bsi_adjoint_workspace_size() is at most BSI_ADJOINT_NOALLOC_MAX_BYTES,
bsi_adjoint_noalloc takes the geometry, so a caller may choose by that size."""
import ctypes
import random

import pytest

from conftest import has_gpu
from paper_2004_05962_amd import _lib

CAP = _lib.BSI_ADJOINT_NOALLOC_MAX_BYTES


@pytest.mark.skipif(has_gpu(), reason="needs the no-device path")
def test_no_geometry_within_the_size_is_refused():
    rng = random.Random(5)
    near = 0
    while near < 3000:
        spacing = [rng.choice([1, 2, 3, 4, 5, 6, 8, 10, 13, 20, 33, 64]) for _ in range(3)]
        dims = [max(1, int(2 ** rng.uniform(2, 11))) for _ in range(3)]
        size = _lib.bsi_adjoint_workspace_size(dims, spacing)
        if not CAP // 2 < size <= CAP:
            continue
        near += 1
        rc = _lib.lib().bsi_adjoint_noalloc(ctypes.c_void_p(256), _lib._triple(dims, "dims"),
                                            _lib._triple(spacing, "spacing"), ctypes.c_void_p(256), ctypes.c_void_p(0))
        # taken: the call ends where it finds no device (the pointers are not followed)
        assert rc == _lib.BSI_ERR_NO_DEVICE, (dims, spacing, size)
