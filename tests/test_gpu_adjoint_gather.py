"""Pass 2 of the adjoint: its workgroup shapes, and partials past its 32-bit offsets.

One point per lane in rows of 16, 32 or 64 points, whichever idles least; a wave
per point where a point has many bricks and the points are few; 64-bit addresses
where the partials exceed 1 GiB.  Bar: max |gpu - oracle| <= 1e-5 * max|oracle
grad|, as for every adjoint here."""
import numpy as np
import pytest
import torch

import oracle
import paper_2004_05962_amd as bsi
import workloads
from gpu_util import dev, host, max_abs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,spacing", [
    ((300, 30, 40), (5, 5, 5)),     # 63 points a row: 64
    ((310, 30, 40), (5, 5, 5)),     # 65: 16 (80 lanes)
    ((460, 20, 40), (5, 5, 5)),     # 95: 32
    ((61, 35, 40), (5, 5, 5)),      # 16 x 10 x 11 points, 3 bricks in y: a wave each
    ((59, 200, 33), (20, 20, 20)),
    ((300, 90, 200), (64, 64, 64)),  # 5 bricks in x, 6 in y, one tile a brick
    ((90, 140, 70), (3, 64, 1)),    # 9 bricks in y
    ((40, 33, 130), (1, 1, 40)),
])
def test_shapes(dims, spacing):
    say("adjoint gather", dims, spacing)
    dfield = workloads.random_field(dims, 1.0, seed=400 + sum(dims))
    got = host(bsi.adjoint(dev(dfield), dims, spacing))
    ref = oracle.adjoint(dfield, dims, spacing)
    assert max_abs(got, ref) <= 1e-5 * float(np.abs(ref).max())


def test_partials_above_one_gibibyte():
    """Spacing 1: each axis is the filter B(0) = (1, 4, 1, 0) / 6, in float64 by
    shifted sums; one volume and a batch of it give the same bits."""
    dims, spacing = (512, 512, 300), (1, 1, 1)
    say("adjoint gather", dims)
    assert bsi.bsi_adjoint_workspace_size(dims, spacing) > 1 << 30
    dfield = torch.randn(bsi.field_shape(dims), device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    got = bsi.adjoint(dfield, dims, spacing)
    ref = dfield.double()
    for axis, n in zip((2, 1, 0), dims):
        shape = list(ref.shape)
        shape[axis] = n + 3
        out = ref.new_zeros(shape)
        for l, w in enumerate((1 / 6, 4 / 6, 1 / 6)):
            out.narrow(axis, l, n).add_(ref, alpha=w)
        ref = out
    assert float((got - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
    del ref
    plan = bsi.BatchPlan([dims], [spacing])
    grad = torch.empty_like(got)
    plan.bind(dfields=[dfield], grid_grads=[grad])
    plan.run()
    assert torch.equal(grad, got)
