"""Edges of the real-spacing adjoint's cells, bricks and gather, and non-finite
upstream values.

Its pass 1 gives a wave up to 32 x 8 voxel columns, fewer below spacing 31 / 12,
where 32 columns meet more than 16 control points.  Bar: max |gpu - oracle| <=
1e-5 * max|oracle grad|, as for every adjoint here; a planted infinity or NaN
makes exactly its window's 4 x 4 x 4 points non-finite."""
import numpy as np
import pytest
import torch

import paper_2004_05962_amd as bsi
from gpu_util import dev, host, max_abs, say
from oracle import general

pytestmark = pytest.mark.gpu

CASES = [
    ((64, 16, 9), (31 / 12, 2.6, 3.3), (-0.5, -1.0, 0.0)),       # cells of 32
    ((65, 17, 20), (2.58, 7.0, 3.3), (-2.5, -6.9, -1.0)),        # just narrower
    ((53, 30, 31), (1.0, 1.0, 1.0), (0.0, -0.5, -0.99)),         # cells of 13, 11 rows, two-plane slabs
    ((27, 9, 60), (1.37, 1.9, 2.2), (-1.3, -0.1, -2.1)),
    ((130, 40, 70), (5.3, 4.7, 5.1), (-5.2, -0.1, -2.5)),
    ((129, 33, 97), (10.0, 9.99, 1.01), (-9.0, 0.0, -0.3)),
    ((200, 90, 50), (40.5, 33.3, 12.1), (-40.0, -1.0, -6.0)),    # a wave per point
    ((31, 7, 1), (64.0, 64.0, 64.0), (-63.5, 0.0, -30.0)),
    ((95, 8, 3), (3.0, 4.0, 5.0), (-2.999, -3.999, -4.999)),
]


def _adjoint(d, dims, spacing, origin):
    out = torch.full(bsi.general_grid_shape(dims, spacing, origin), float("nan"), device="cuda")
    nbytes = bsi.bsi_adjoint_general_workspace_size(dims, spacing, origin)
    ws = torch.full((nbytes + 1024,), 0xFF, dtype=torch.uint8, device="cuda")
    bsi.bsi_adjoint_general(dev(d), dims, spacing, origin, out, ws[:nbytes])
    assert bool((ws[nbytes:] == 0xFF).all()), "wrote past the workspace"
    return host(out)


@pytest.mark.parametrize("dims,spacing,origin", CASES)
def test_cell_edges(dims, spacing, origin):
    say("general cells", dims, spacing, origin)
    nx, ny, nz = dims
    d = np.random.default_rng(nx + ny).standard_normal((nz, ny, nx, 3)).astype(np.float32)
    ref = general.adjoint(d, dims, spacing, origin)
    assert max_abs(_adjoint(d, dims, spacing, origin), ref) <= 1e-5 * float(np.abs(ref).max())


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_non_finite_values_reach_their_window_only(value):
    dims, spacing, origin = (70, 20, 22), (4.5, 3.25, 5.0), (-2.0, 0.0, -1.25)
    say("general non-finite", value)
    d = np.random.default_rng(8).standard_normal((22, 20, 70, 3)).astype(np.float32)
    clean = general.adjoint(d, dims, spacing, origin)
    hit = np.zeros(clean.shape, dtype=bool)
    for c, v in enumerate([(33, 9, 11), (5, 19, 0), (69, 0, 21)]):  # the last on a control row: a zero weight
        d[v[2], v[1], v[0], c] = value
        t = [int(np.floor((x - o) / s)) for x, s, o in zip(v, spacing, origin)]
        hit[t[2]:t[2] + 4, t[1]:t[1] + 4, t[0]:t[0] + 4, c] = True
    got = _adjoint(d, dims, spacing, origin)
    assert np.array_equal(~np.isfinite(got), hit)
    assert max_abs(got[~hit], clean[~hit]) <= 1e-5 * float(np.abs(clean).max())
