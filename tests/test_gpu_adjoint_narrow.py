"""Adjoint with cells of at most 16 columns (16 lanes a row): widths on and beside the
cells' limits, both ways of keeping the slabs, aligned, real-spacing and batched.

Bar: max |gpu - oracle| <= 1e-5 * max|oracle grad|, as for every adjoint here; a batched
volume has the bits of the single call."""
import numpy as np
import pytest
import torch

import oracle
import paper_2004_05962_amd as bsi
import workloads
from gpu_util import dev, host, max_abs, say
from oracle import general as ogen

pytestmark = pytest.mark.gpu

EDGES = [
    ((13, 8, 20), (1, 1, 1)),
    ((25, 9, 7), (1, 1, 1)),
    ((26, 16, 40), (1, 1, 1)),
    ((27, 17, 33), (1, 1, 1)),
    ((53, 33, 61), (1, 2, 1)),
    ((40, 40, 21), (1, 8, 5)),     # windows of 5 rows: shared products
    ((40, 40, 21), (1, 2, 3)),     # of 8 rows
    ((31, 20, 19), (2, 2, 2)),     # cells of 16 columns
    ((32, 20, 19), (2, 1, 1)),
    ((33, 20, 19), (2, 2, 2)),     # of 18: not narrow
    ((300, 64, 130), (1, 1, 1)),   # two-plane slabs
    ((1, 300, 40), (1, 1, 1)),
    ((5, 3, 2), (3, 3, 3)),
]


@pytest.mark.parametrize("dims,spacing", EDGES)
def test_narrow_cells(dims, spacing):
    say("adjoint narrow", dims, spacing)
    dfield = workloads.random_field(dims, 1.0, seed=400 + sum(dims))
    got = host(bsi.adjoint(dev(dfield), dims, spacing))
    ref = oracle.adjoint(dfield, dims, spacing)
    assert max_abs(got, ref) <= 1e-5 * float(np.abs(ref).max())
    # beside a wide volume, so that one plan holds narrow and whole cells
    plan = bsi.BatchPlan([dims, (70, 20, 15)], [spacing, (5, 5, 5)])
    grids = [torch.zeros(bsi.grid_shape(d, s), device="cuda") for d, s in ((dims, spacing), ((70, 20, 15), (5, 5, 5)))]
    fields = [torch.empty(bsi.field_shape(d), device="cuda") for d in (dims, (70, 20, 15))]
    grads = [torch.full_like(g, float("nan")) for g in grids]
    plan.bind(grids, fields, [dev(dfield), torch.zeros_like(fields[1])], grads)
    plan.run()
    torch.cuda.synchronize()
    assert np.array_equal(host(grads[0]), got)
    plan.close()


@pytest.mark.parametrize("dims,spacing,origin", [
    ((26, 23, 40), (1.0, 1.0, 1.0), (0.0, 0.0, 0.0)),
    ((33, 19, 21), (1.25, 1.5, 1.1), (-1.0, -0.3, -0.5)),   # cells of 16 and 17 columns
    ((200, 70, 90), (1.3, 1.0, 1.2), (-0.2, 0.0, -1.1)),
    ((60, 40, 30), (1.1, 9.5, 3.5), (-1.0, -4.0, 0.0)),
])
def test_narrow_cells_real_spacing(dims, spacing, origin):
    say("general adjoint narrow", dims, spacing, origin)
    dfield = workloads.random_field(dims, 1.0, seed=3 + sum(dims))
    grad = torch.empty(bsi.general_grid_shape(dims, spacing, origin), device="cuda")
    ws = torch.empty(bsi.bsi_adjoint_general_workspace_size(dims, spacing, origin), dtype=torch.uint8, device="cuda")
    bsi.bsi_adjoint_general(dev(dfield), dims, spacing, origin, grad, ws)
    ref = ogen.adjoint(dfield, dims, spacing, origin)
    assert max_abs(host(grad), ref) <= 1e-5 * float(np.abs(ref).max())


@pytest.mark.parametrize("dims,spacing", [((34, 6200, 33), (2, 1, 1)), ((55, 7000, 32), (1, 10, 1)),
                                          ((991, 885, 107), (1, 20, 12))])
def test_noalloc_with_the_largest_partials(dims, spacing):
    """Partials of up to 1.24 times the limit's size, in the fixed scratch: the bits of
    bsi_adjoint, whose workspace is followed by a guard."""
    say("adjoint noalloc, largest partials", dims, spacing)
    dfield = torch.randn(bsi.field_shape(dims), device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    nbytes = bsi.bsi_adjoint_workspace_size(dims, spacing)
    ws = torch.full((nbytes + 1024,), 0xFF, dtype=torch.uint8, device="cuda")
    expect = torch.empty(bsi.grid_shape(dims, spacing), device="cuda")
    bsi.bsi_adjoint(dfield, dims, spacing, expect, ws[:nbytes])
    got = torch.full_like(expect, float("nan"))
    bsi.bsi_adjoint_noalloc(dfield, dims, spacing, got)
    torch.cuda.synchronize()
    assert torch.equal(got, expect)
    assert bool((ws[nbytes:] == 0xFF).all())
    # the transpose identity <A g, d> = <g, A^T d>, in FP64 sums of FP32 values
    grid = torch.randn(expect.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(4))
    field = bsi.forward(grid, dims, spacing).double()
    a, b = float((field * dfield).sum()), float((grid.double() * got).sum())
    scale = float(field.square().sum().sqrt() * dfield.double().square().sum().sqrt())
    assert abs(a - b) <= 1e-6 * scale
