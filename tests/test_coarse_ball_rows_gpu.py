"""Coarse bounds with a ball on rows that are not whole 16-byte groups, and on rows shorter than
one: rows of cells that the ball reaches hold the full bound bit for bit, those out of its
reach -inf, whatever the table held before (a stale finite bound there would let a later plan
step skip lookups)."""
import numpy as np
import pytest

from synth import workload as W
from tests.test_coarse_gpu import cells_reached, coarse_reference

pytestmark = pytest.mark.gpu

STALE = 7.0


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("nx", [2, 3, 7, 25, 150, 499])
def test_rows_out_of_reach(nx, f16):
    import torch

    from paper_2512_22575_amd import smpc as S
    rng = np.random.default_rng(nx + f16)
    grid = np.clip(rng.normal(scale=0.3, size=(40, 41, nx)), -2, 2).astype(np.float32)
    grid[3, 5, nx - 1] = np.inf
    if f16:
        grid = grid.astype(np.float16)
    origin, voxel = W.f32([-0.4, -0.3, 0.1]), W.f32s(0.01)
    extent = np.array(grid.shape[::-1]) * voxel
    center = W.f32(origin + extent * np.array([0.2, 0.6, 0.5]))
    radius = float(0.3 * extent[1:].min())
    full = coarse_reference(grid.astype(np.float32))
    bits = torch.from_numpy(grid.view(np.int16) if f16 else grid).cuda()
    out = torch.full((full.size,), STALE, device="cuda")
    st = S.smpc_grid_coarse_min_ball(bits, S.GRID_F16 if f16 else S.GRID_F32, origin, voxel, center,
                                     radius, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == S.SMPC_OK
    got = out.cpu().numpy().reshape(full.shape)
    # The library widens the ball by one voxel, so that it covers a lookup's float32 rounding.
    inside = cells_reached(grid.shape, origin, voxel, center, radius).any(axis=2)
    beyond = ~cells_reached(grid.shape, origin, voxel, center, radius + 1.001 * voxel).any(axis=2)
    assert inside.any() and beyond.any()
    assert np.array_equal(got[inside].view(np.uint32), full[inside].view(np.uint32))
    assert np.all(got[beyond] == -np.inf)
