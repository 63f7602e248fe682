"""Fused SSD step with an infinity or a NaN in an image: bit-identical to the separate
forward, SSD and adjoint, also in the finite points of the planes that hold one.

The planted voxel lies beside a cell's border, in narrow cells (x spacings 1 and 2) and
whole ones: what a cell sums does not depend on its neighbour's voxels."""
import numpy as np
import pytest
import torch

import paper_2004_05962_amd as bsi
from gpu_util import host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,spacing,voxel", [
    ((60, 20, 14), (1, 1, 1), (10, 3, 5)),   # cells of 10 columns
    ((60, 20, 14), (1, 1, 1), (9, 8, 5)),
    ((100, 20, 14), (2, 2, 2), (26, 3, 6)),  # of 18
    ((90, 40, 21), (5, 5, 5), (32, 8, 7)),
    ((90, 40, 21), (5, 5, 5), (31, 15, 20)),
])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_fused_with_non_finite_voxel_equals_separate(dims, spacing, voxel, value):
    say("fused non-finite", dims, spacing, voxel, value)
    gen = torch.Generator(device="cuda").manual_seed(5)
    shape = tuple(reversed(dims))
    grid = torch.rand(bsi.grid_shape(dims, spacing), device="cuda", generator=gen) - 0.5
    moving = torch.rand(shape, device="cuda", generator=gen)
    fixed = torch.rand(shape, device="cuda", generator=gen)
    fixed[voxel[2], voxel[1], voxel[0]] = value

    field = bsi.forward(grid, dims, spacing)
    dT = torch.empty_like(field)
    loss = torch.empty(1, device="cuda")
    bsi.bsi_ssd_grad(field, moving, fixed, dims, dT, loss,
                     torch.empty(bsi.bsi_ssd_workspace_size(dims), dtype=torch.uint8, device="cuda"))
    expect = host(bsi.adjoint(dT, dims, spacing))
    got = torch.empty(expect.shape, device="cuda")
    fused_loss = torch.empty(1, device="cuda")
    bsi.bsi_ssd_fused(grid, moving, fixed, dims, spacing, got, fused_loss,
                      torch.empty(bsi.bsi_ssd_fused_workspace_size(dims, spacing), dtype=torch.uint8, device="cuda"))
    assert (~np.isfinite(expect)).sum() == 192
    assert np.array_equal(host(got), expect, equal_nan=True)
    assert not np.isfinite(float(fused_loss)) and not np.isfinite(float(loss))
