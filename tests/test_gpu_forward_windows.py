"""The forward's workgroup shapes and window sizes at the limits between them.

A window is sized for the smallest x and y spacing of its instance (vector 1, 3,
5; scalar 1, 2, 4 with four voxels per lane and 1, 2, 3 with one; real spacing
1 and 3), and holds the most control columns where a tile begins one voxel
before the strip does.  Bar: max |gpu - oracle| <= 1e-5 * max|grid|, as for every
forward here."""
import itertools

import numpy as np
import pytest
import torch

import oracle
import paper_2004_05962_amd as bsi
import workloads
from gpu_util import dev, host, max_abs, say
from oracle import general, scalar

pytestmark = pytest.mark.gpu

PAIRS = [(1, 1), (2, 3), (3, 2), (3, 3), (4, 5), (5, 4), (5, 5), (6, 9)]


# rows on 64-byte boundaries (one strip; whole rows and a ragged second
# workgroup), off them, and z-chunks that end inside a tile
@pytest.mark.parametrize("dxy,nx,dz", [(p, nx, dz) for p, (nx, dz) in itertools.product(
    PAIRS, [(144, 4), (528, 5), (272, 31), (131, 7)])])
def test_vector(dxy, nx, dz):
    dims, spacing = (nx, 7, 65), (*dxy, dz)
    say("forward windows", dims, spacing)
    grid = workloads.random_grid(dims, spacing, 2.0, seed=nx + 10 * dxy[0] + dxy[1])
    got = host(bsi.forward(dev(grid), dims, spacing))
    assert max_abs(got, oracle.forward(grid, dims, spacing)) <= 1e-5 * float(np.abs(grid).max())


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("nx", [516, 131])
def test_scalar(d, nx):
    dims, spacing = (nx, 10, 9), (d, d, 3)
    say("scalar windows", dims, spacing)
    gx, gy, gz = bsi.bsi_grid_dims(dims, spacing)
    grid = np.random.default_rng(d).standard_normal((gz, gy, gx)).astype(np.float32)
    out = torch.empty((9, 10, nx), device="cuda")
    bsi.bsi_forward_scalar(dev(grid), dims, spacing, out)
    assert max_abs(host(out), scalar.forward(grid, dims, spacing)) <= 1e-5 * float(np.abs(grid).max())


@pytest.mark.parametrize("s", [np.nextafter(np.float32(3), np.float32(0)), 3.0, np.nextafter(np.float32(3), np.float32(4))])
@pytest.mark.parametrize("nx", [192, 130])
def test_real_spacing(s, nx):
    dims, spacing, origin = (nx, 9, 20), (float(s), float(s), 2.5), (-1.0, -2.0, -0.5)
    say("general forward windows", dims, spacing)
    gx, gy, gz = bsi.bsi_general_grid_dims(dims, spacing, origin)
    grid = np.random.default_rng(nx).standard_normal((gz, gy, gx, 3)).astype(np.float32)
    out = torch.empty(bsi.field_shape(dims), device="cuda")
    bsi.bsi_forward_general(dev(grid), dims, spacing, origin, out)
    assert max_abs(host(out), general.forward(grid, dims, spacing, origin)) <= 1e-5 * float(np.abs(grid).max())


@pytest.mark.parametrize("least", [1, 3, 5])
def test_batch_of_one_least_spacing(least):
    geoms = [((140, 9, 33), (least, 7, 5)), ((64, 30, 7), (6, least, 9)), ((77, 8, 20), (8, 5, 3))]
    say("batch windows", least)
    grids = [workloads.random_grid(d, s, 2.0, seed=i) for i, (d, s) in enumerate(geoms)]
    fields = [torch.empty(bsi.field_shape(d), device="cuda") for d, _ in geoms]
    bound = [dev(g) for g in grids]
    plan = bsi.BatchPlan([d for d, _ in geoms], [s for _, s in geoms])
    plan.bind(grids=bound, fields=fields)
    plan.run()
    for (d, s), g, f in zip(geoms, grids, fields):
        assert max_abs(host(f), oracle.forward(g, d, s)) <= 1e-5 * float(np.abs(g).max())
