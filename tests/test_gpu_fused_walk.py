"""Fused SSD step over several z-tiles and z-bricks per workgroup, on random grids.

The fused pass performs the operations of the separate forward, SSD and adjoint
kernels in their order, so the control-grid gradient is bit-identical to theirs.
The sizes take more than one z-tile (the ring of staged control planes is refilled),
more than one z-brick per workgroup, a partial last tile, two-plane slabs, several
staged loads per thread (spacing 1) and a volume one voxel wide.
Loss bar: 1e-5 relative to the FP64 sum of the squared FP32 residuals."""
import pytest
import torch

import paper_2004_05962_amd as bsi
from gpu_util import say

pytestmark = pytest.mark.gpu

CASES = [
    ((256, 256, 160), (5, 5, 5)),
    ((512, 300, 199), (5, 5, 5)),
    ((1024, 260, 210), (5, 5, 5)),
    ((512, 510, 199), (5, 5, 5)),
    ((200, 220, 240), (2, 3, 1)),
    ((300, 260, 40), (5, 5, 1)),
    ((64, 64, 200), (1, 1, 1)),
    ((300, 256, 200), (1, 1, 1)),
    ((1, 40, 50), (3, 3, 3)),
    ((100, 50, 90), (2, 2, 2)),
    ((130, 33, 129), (2, 3, 64)),
    ((97, 40, 41), (2, 1, 3)),
    ((59, 35, 23), (1, 4, 5)),
    ((31, 20, 40), (2, 2, 1)),
]


@pytest.mark.parametrize("dims,spacing", CASES)
def test_fused_equals_forward_ssd_adjoint(dims, spacing):
    say("fused walk", dims, spacing)
    gen = torch.Generator(device="cuda").manual_seed(17 + sum(dims))
    shape = tuple(reversed(dims))
    grid = torch.rand(bsi.grid_shape(dims, spacing), device="cuda", generator=gen) * 4 - 2
    moving = torch.rand(shape, device="cuda", generator=gen)
    fixed = torch.rand(shape, device="cuda", generator=gen)

    field = bsi.forward(grid, dims, spacing)
    dT = torch.empty_like(field)
    loss = torch.empty(1, device="cuda")
    bsi.bsi_ssd_grad(field, moving, fixed, dims, dT, loss,
                     torch.empty(bsi.bsi_ssd_workspace_size(dims), dtype=torch.uint8, device="cuda"))
    expect = bsi.adjoint(dT, dims, spacing)
    warped = torch.empty(shape, device="cuda")
    bsi.bsi_warp(field, moving, dims, warped)
    total = float((warped - fixed).double().square().sum())

    ws = torch.empty(bsi.bsi_ssd_fused_workspace_size(dims, spacing), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        got = torch.full_like(expect, float("nan"))
        fused_loss = torch.full((1,), float("nan"), device="cuda")
        bsi.bsi_ssd_fused(grid, moving, fixed, dims, spacing, got, fused_loss, ws)
        torch.cuda.synchronize()
        assert torch.equal(got, expect)
        assert abs(float(fused_loss) - total) <= 1e-5 * total
    assert abs(float(loss) - total) <= 1e-5 * total
