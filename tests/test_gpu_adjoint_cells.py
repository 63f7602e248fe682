"""Edges of the adjoint's cells and bricks, and non-finite upstream values.

Pass 1 gives a wave 32 x 8 voxel columns (13 x 8 at x spacing 1, 24 x 8 at 2), two
by two cells a workgroup, and contracts them on 16 x 16 matrix tiles; windows
of at most 5 and 8 rows share products, and bricks whose slabs do not fit the LDS
take two-plane slabs.  The sizes below sit on and beside each of these limits.

Bar: max |gpu - oracle| <= 1e-5 * max|oracle grad|, as for every adjoint here.
For a planted infinity or NaN: exactly the 4 x 4 x 4 control points of its
voxel's window are non-finite, the others are those of the field without it,
within 1e-5 (the infinite plane is summed in another order)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2004_05962_amd as bsi
import workloads
from gpu_util import dev, host, max_abs, say

pytestmark = pytest.mark.gpu

EDGES = [
    ((32, 8, 5), (3, 3, 3)),      # one cell, whole
    ((33, 9, 6), (3, 3, 3)),      # one voxel into the next cell and row
    ((31, 7, 1), (5, 5, 5)),      # one plane
    ((64, 16, 2), (5, 5, 5)),     # one brick, two planes
    ((65, 17, 3), (5, 5, 5)),
    ((63, 15, 97), (6, 6, 6)),    # windows of 5 rows; more than one brick deep
    ((26, 16, 31), (1, 1, 1)),    # spacing 1: two cells of 13, two-plane slabs, one plane past a brick
    ((27, 17, 30), (1, 1, 1)),
    ((14, 23, 9), (1, 1, 4)),
    ((48, 24, 50), (2, 2, 2)),    # spacing 2: cells of 24
    ((49, 25, 17), (2, 2, 2)),
    ((50, 9, 40), (2, 1, 3)),     # 11 rows: no shared products
    ((70, 40, 33), (7, 7, 1)),    # a z-tile per plane, two-plane slabs
    ((96, 33, 65), (32, 8, 16)),
    ((130, 18, 70), (64, 64, 64)),
    ((129, 31, 20), (4, 2, 3)),
]


@pytest.mark.parametrize("dims,spacing", EDGES)
def test_cell_edges(dims, spacing):
    say("adjoint cells", dims, spacing)
    dfield = workloads.random_field(dims, 1.0, seed=900 + sum(dims))
    got = host(bsi.adjoint(dev(dfield), dims, spacing))
    ref = oracle.adjoint(dfield, dims, spacing)
    assert max_abs(got, ref) <= 1e-5 * float(np.abs(ref).max())


@pytest.mark.parametrize("dims,spacing", [((70, 20, 22), (5, 5, 5)), ((40, 12, 9), (3, 4, 2)), ((30, 18, 7), (1, 1, 1)),
                                          ((50, 33, 40), (13, 9, 6))])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_non_finite_values_reach_their_window_only(dims, spacing, value):
    say("adjoint non-finite", dims, spacing, value)
    rng = np.random.default_rng(77)
    dfield = workloads.random_field(dims, 1.0, seed=31)
    clean = oracle.adjoint(dfield, dims, spacing)
    hit = np.zeros(clean.shape, dtype=bool)
    for c in range(3):  # one voxel per component, the first at offset 0 of its tile
        v = [int(rng.integers(0, n)) for n in dims]
        if c == 0:
            v = [(x // d) * d for x, d in zip(v, spacing)]
        dfield[v[2], v[1], v[0], c] = value
        t = [x // d for x, d in zip(v, spacing)]
        hit[t[2]:t[2] + 4, t[1]:t[1] + 4, t[0]:t[0] + 4, c] = True
    got = host(bsi.adjoint(dev(dfield), dims, spacing))
    assert np.array_equal(~np.isfinite(got), hit)
    assert max_abs(got[~hit], clean[~hit]) <= 1e-5 * float(np.abs(clean).max())
