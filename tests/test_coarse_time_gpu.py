"""Coarse bounds of rows that are not whole 16-byte groups take about as long as those of whole
ones: the same rows are loaded and folded, a wave's loads spanning one 128-byte line more at
most, and the columns that two groups share are sorted out once per group and not per row.
Half as much again is allowed."""
import numpy as np
import pytest

from synth import workload as W

pytestmark = pytest.mark.gpu


def _us(nx, f16, ball):
    import torch

    from paper_2512_22575_amd import smpc as S
    grid = torch.rand((400, 400, nx), device="cuda").to(torch.float16 if f16 else torch.float32)
    dtype = S.GRID_F16 if f16 else S.GRID_F32
    out = torch.empty(S.smpc_grid_coarse_cells(nx, 400, 400), device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    origin, center = W.f32([-1.0, -1.0, 0.0]), W.f32([0.0, 0.0, 0.3])

    def call():
        if ball:
            return S.smpc_grid_coarse_min_ball(grid, dtype, origin, W.f32s(0.005), center, 0.6,
                                               out.data_ptr(), stream)
        return S.smpc_grid_coarse_min(grid, dtype, out.data_ptr(), stream)

    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    times = []
    for _ in range(9):
        a.record()
        for _ in range(50):
            assert call() == S.SMPC_OK
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / 50)
    return float(np.median(times))


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("ball", [False, True])
def test_ragged_rows_cost_what_whole_ones_do(f16, ball):
    ragged, whole = _us(25, f16, ball), _us(24, f16, ball)
    print(f"f16 {f16} ball {ball}: 25 columns {ragged:.1f} us, 24 columns {whole:.1f} us", flush=True)
    assert ragged <= 1.5 * whole
