"""The warp and SSD kernels where their columns and z-chunks can go wrong: rows
that end inside a wave, planes that end inside a block of 256 columns, chunks of
an odd number of planes, axes of one voxel, images of 4 GiB and more.

Bar (as the registration tests): values within 1e-5 of the image range, the field
gradient within 1e-5 of its largest value, the loss within 1e-5 relative, against
the FP64 oracle with the sample coordinate formed in FP32."""
import numpy as np
import pytest
import torch

import paper_2004_05962_amd as bsi
from gpu_util import dev, host, max_abs, say
from oracle import warp as owarp

pytestmark = pytest.mark.gpu

SHAPES = [  # (nz, ny, nx)
    (1, 1, 1), (1, 1, 300), (1, 257, 1), (131, 1, 1), (5, 16, 16), (9, 17, 15), (4, 16, 16),
    (3, 85, 3), (33, 20, 39), (2, 130, 67), (70, 3, 511), (257, 2, 2),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_columns_and_chunks(shape):
    nz, ny, nx = shape
    dims = (nx, ny, nz)
    say("sampling", dims)
    rng = np.random.default_rng(sum(shape))
    moving = rng.standard_normal(shape).astype(np.float32)
    fixed = rng.standard_normal(shape).astype(np.float32)
    field = (rng.standard_normal(shape + (3,)) * 2.5).astype(np.float32)
    F, M, X = dev(field), dev(moving), dev(fixed)
    W = torch.full(shape, float("nan"), device="cuda")
    bsi.bsi_warp(F, M, dims, W)
    scale = float(np.abs(moving).max())
    assert max_abs(host(W), owarp.warp(moving, field, coord_dtype=np.float32)) <= 1e-5 * scale
    dT = torch.full(shape + (3,), float("nan"), device="cuda")
    loss = torch.full((1,), float("nan"), device="cuda")
    ws = torch.empty(bsi.bsi_ssd_workspace_size(dims), dtype=torch.uint8, device="cuda")
    bsi.bsi_ssd_grad(F, M, X, dims, dT, loss, ws)
    L_ref, dT_ref = owarp.ssd_grad(field, moving, fixed, coord_dtype=np.float32)
    assert max_abs(host(dT), dT_ref) <= 1e-5 * max(float(np.abs(dT_ref).max()), 1e-30)
    assert abs(float(host(loss)[0]) - L_ref) <= 1e-5 * L_ref


def test_image_beyond_buffer_offsets():
    """An image of 4 GiB + 4 MiB: corners addressed with 64 bits; checked at sampled voxels."""
    dims = (1024, 1024, 1025)
    say("sampling", dims)
    nx, ny, nz = dims
    gen = torch.Generator(device="cuda").manual_seed(3)
    image = torch.randn((nz, ny, nx), generator=gen, device="cuda")
    field = torch.randn((nz, ny, nx, 3), generator=gen, device="cuda") * 2.0
    out = torch.empty_like(image)
    bsi.bsi_warp(field, image, dims, out)
    n = 4000
    v = [torch.randint(0, m, (n,), generator=gen, device="cuda") for m in (nz, ny, nx)]
    v[0][:500] = nz - 1 - torch.arange(500, device="cuda") % 4
    t = field[v[0], v[1], v[2]]
    want, lo, fr = torch.zeros(n, dtype=torch.float64, device="cuda"), [], []
    for k, m in enumerate((nz, ny, nx)):
        p = (v[k].float() + t[:, 2 - k]).clamp(0, m - 1).double()
        i = torch.floor(p).clamp(max=m - 2)
        lo.append(i.long())
        fr.append(p - i)
    for c in range(8):
        b = [(c >> k) & 1 for k in range(3)]
        w = [fr[k] if b[k] else 1 - fr[k] for k in range(3)]
        want += image[lo[0] + b[0], lo[1] + b[1], lo[2] + b[2]].double() * w[0] * w[1] * w[2]
    got = out[v[0], v[1], v[2]].double()
    assert float((got - want).abs().max()) <= 1e-5 * float(image.abs().max())
