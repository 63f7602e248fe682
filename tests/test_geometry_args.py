"""Geometry arguments of the Python layer, whose results are kept by value: any
sequence of three numbers, the same answer from every form of them, and an error
on every call for an invalid one."""
import numpy as np
import pytest

import paper_2004_05962_amd as bsi
from paper_2004_05962_amd import _lib


@pytest.mark.parametrize("form", [tuple, list, np.array, lambda v: np.array(v, dtype=np.int16), lambda v: [float(x) for x in v]])
def test_forms(form):
    dims, spacing = (33, 64, 7), (5, 3, 64)
    assert bsi.bsi_grid_dims(form(dims), form(spacing)) == (10, 25, 4)
    assert bsi.grid_shape(form(dims), form(spacing)) == (4, 25, 10, 3)
    assert bsi.field_shape(form(dims)) == (7, 64, 33, 3)
    assert bsi.bsi_adjoint_workspace_size(form(dims), form(spacing)) == bsi.bsi_adjoint_workspace_size(dims, spacing)


def test_errors_on_every_call():
    for _ in range(2):
        for f in (bsi.bsi_grid_dims, bsi.grid_shape, bsi.bsi_adjoint_workspace_size):
            with pytest.raises(ValueError):
                f((1, 2), (1, 1, 1))
            with pytest.raises(_lib.BSIError) as e:
                f((4, 4, 4), (1, 0, 1))
            assert e.value.code == _lib.BSI_ERR_INVALID_ARG and "spacing" in str(e.value)
