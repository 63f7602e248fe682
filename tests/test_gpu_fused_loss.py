"""The fused step's loss at many planes: its FP32 sums form chains whose length does not
grow with the volume.

Every residual is 0.9, so the exact loss is known.  A lane sums the squares of one
z-brick's planes (at most 96) in one chain, its bricks' sums in another, the workgroup
its 1024 lanes in a tree of 10, and the tail the partials (one per thread here) in a
tree of 8.  All terms are positive: a term passes through at most
96 + bricks + 10 + 8 + 1 roundings of 2^-24 each, which is the bar.  One chain over
all of a column's 2000 planes is off by 2.5e-5."""
import ctypes
import os

import numpy as np
import pytest
import torch

import paper_2004_05962_amd as bsi
from conftest import ROOT
from gpu_util import say

pytestmark = pytest.mark.gpu


def test_fused_loss_over_many_planes():
    dims, spacing = (2, 4096, 2000), (5, 5, 5)
    say("fused loss", dims, spacing)
    info = (ctypes.c_int32 * 2)()
    msg = ctypes.create_string_buffer(512)
    L = ctypes.CDLL(os.path.join(ROOT, "paper_2004_05962_amd", "libbsi_check.so"))
    assert L.bsi_check_fused((ctypes.c_int32 * 3)(*dims), (ctypes.c_int32 * 3)(*spacing), info, msg, 512) == 0
    bricks = info[0]
    assert 2000 / 96 <= bricks <= 50  # every z-brick of a column in one workgroup
    shape = tuple(reversed(dims))
    grid = torch.zeros(bsi.grid_shape(dims, spacing), device="cuda")
    moving = torch.zeros(shape, device="cuda")
    fixed = torch.full(shape, 0.9, device="cuda")
    got = torch.empty_like(grid)
    loss = torch.empty(1, device="cuda")
    bsi.bsi_ssd_fused(grid, moving, fixed, dims, spacing, got, loss,
                      torch.empty(bsi.bsi_ssd_fused_workspace_size(dims, spacing), dtype=torch.uint8, device="cuda"))
    exact = float(np.float32(0.9)) ** 2 * np.prod(dims)
    rel = abs(float(loss) - exact) / exact
    say(f"  loss rel {rel:.2e}")
    assert rel <= (96 + bricks + 10 + 8 + 1) * 2.0 ** -24
