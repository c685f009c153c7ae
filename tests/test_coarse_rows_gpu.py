"""Coarse lower bounds of grids whose rows are not whole 16-byte groups, or that do not start on
a 16-byte boundary, at the row lengths where the last group, the last window or the number
of chunks changes: bit for bit their definition; and with a ball, whole rows of cells, full
or -inf."""
import numpy as np
import pytest

from synth import workload as W
from tests.test_coarse_gpu import cells_reached, coarse_reference, gpu_coarse, gpu_coarse_ball

pytestmark = pytest.mark.gpu


def _on_device(g, off):
    """g on the device, `off` elements into its buffer, whose last element is g's."""
    import torch
    bits = torch.from_numpy(g.view(np.int16 if g.dtype == np.float16 else np.int32).reshape(-1))
    buf = torch.zeros(off + g.size, dtype=bits.dtype, device="cuda")
    buf[off:] = bits.cuda()
    return buf[off:].view(g.shape)


@pytest.mark.parametrize("nx", [2, 3, 4, 5, 6, 7, 8, 9, 10, 15, 16, 17, 18, 25, 150, 247, 248, 249,
                                250, 253, 497, 504, 505, 506, 513])
@pytest.mark.parametrize("off", [0, 1, 3])
def test_row_lengths(nx, off):
    from paper_2512_22575_amd import smpc as S
    rng = np.random.default_rng(nx + 1000 * off)
    grid = rng.normal(scale=0.3, size=(11, 10, nx)).astype(np.float32)
    if nx > 20:
        grid[3, 4, nx - 1] = np.nan
        grid[10, 9, nx - 3] = np.inf
        grid[0, 0, nx // 2] = -np.inf
    g16 = np.clip(grid, -2, 2).astype(np.float16)
    for g, dtype in ((grid, S.GRID_F32), (g16, S.GRID_F16)):
        got = gpu_coarse(_on_device(g, off), dtype).cpu().numpy()
        want = coarse_reference(g.astype(np.float32)).reshape(-1)
        np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("nx", [150, 499])
def test_ball(nx):
    from paper_2512_22575_amd import smpc as S
    rng = np.random.default_rng(nx)
    grid = rng.normal(scale=0.3, size=(40, 41, nx)).astype(np.float32)
    origin, voxel = W.f32([-0.4, -0.3, 0.1]), W.f32s(0.01)
    extent = np.array(grid.shape[::-1]) * voxel
    center = W.f32(origin + extent * np.array([0.2, 0.6, 0.5]))
    radius = float(0.3 * extent.min())
    full = coarse_reference(grid)
    rows = cells_reached(grid.shape, origin, voxel, center, radius).any(axis=2)
    assert 0 < rows.sum() < rows.size
    got = gpu_coarse_ball(_on_device(grid, 0), S.GRID_F32, origin, voxel, center, radius)
    got = got.cpu().numpy().reshape(full.shape)
    assert np.array_equal(got[rows].view(np.uint32), full[rows].view(np.uint32))
