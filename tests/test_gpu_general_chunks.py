"""Real-spacing forward at the depths of its z-chunks: rows on and off 64-byte boundaries,
up to the 256 planes that a workgroup's table of z weights holds (4 tiles of 64).

Bar: max |gpu - oracle| <= 1e-5 * max|grid|, as for every forward here."""
import numpy as np
import pytest
import torch

import paper_2004_05962_amd as bsi
from gpu_util import dev, host, max_abs, say
from oracle import general

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,spacing,origin", [
    ((65, 9, 600), (3.3, 4.4, 64.0), (-1.0, 0.0, -20.0)),
    ((65, 9, 257), (3.3, 1.4, 63.9), (-1.0, 0.0, 0.0)),
    ((64, 9, 600), (3.3, 4.4, 64.0), (-1.0, 0.0, -20.0)),
    ((70, 130, 101), (13.46, 1.59, 10.34), (-3.0, -0.5, -2.0)),
    ((33, 260, 151), (2.0, 5.1, 12.5), (0.0, -5.0, -12.0)),
    ((31, 40, 103), (4.5, 4.5, 3.9), (-4.0, 0.0, -1.0)),
    ((80, 40, 149), (2.5, 1.5, 2.2), (-1.0, 0.0, -2.0)),
])
def test_general_forward_chunks(dims, spacing, origin):
    say("general forward chunks", dims, spacing, origin)
    rng = np.random.default_rng(sum(dims))
    grid = rng.standard_normal(bsi.general_grid_shape(dims, spacing, origin)).astype(np.float32)
    field = torch.full(bsi.field_shape(dims), float("nan"), device="cuda")
    bsi.bsi_forward_general(dev(grid), dims, spacing, origin, field)
    ref = general.forward(grid, dims, spacing, origin)
    assert max_abs(host(field), ref) <= 1e-5 * float(np.abs(grid).max())
