"""The x pass of the distance field (16 lanes per row, 16 voxels per lane for rows of up to
256 voxels, 24 up to 384, 32 for longer ones) at the row lengths where a lane, the last lane's stores or
the voxels per lane change, with occupancy bytes of any non-zero value, the grid starting
at any byte and ending with its buffer's data.  Every result is an integer, so the bound
is equality."""
import numpy as np
import pytest

from oracle import edt as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [1, 2, 3, 7, 8, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 127,
                                240, 241, 255, 256, 257, 271, 272, 287, 288, 289, 333, 360,
                                383, 384, 385, 496, 497, 511,
                                512])
def test_row_lengths(nx):
    import torch

    from paper_2512_22575_amd import smpc as S
    ny, nz = 3, 7     # 21 rows: a block of 16 and a part of one
    rng = np.random.default_rng(nx)
    dev = torch.device("cuda:0")
    for off, density in ((0, 0.03), (1, 0.97), (3, 0.4), (7, 0.01)):
        occ = rng.uniform(size=(nz, ny, nx)) < density
        occ[0, 0], occ[0, 1] = False, True                  # a row of each kind only
        occ[0, 2], occ[1, 0] = False, True
        occ[0, 2, -1], occ[1, 0, 0] = True, False           # one voxel of the other at an end
        grid = np.where(occ, rng.choice([1, 2, 0x40, 0x80, 0xFF], size=occ.shape), 0)
        buf = torch.full((off + occ.size + 64,), 255, dtype=torch.uint8, device=dev)
        buf[off:off + occ.size] = torch.from_numpy(grid.astype(np.uint8).reshape(-1)).to(dev)
        need = S.smpc_edt_workspace_bytes(nx, ny, nz)
        work = torch.full((need,), 255, dtype=torch.uint8, device=dev)
        d2 = torch.full((2,) + occ.shape, -1, dtype=torch.int32, device=dev)
        st = S.smpc_edt(buf.data_ptr() + off, nx, ny, nz, 0.02, None, d2.data_ptr(),
                        work.data_ptr(), need, torch.cuda.current_stream().cuda_stream)
        assert st == S.SMPC_OK, S.smpc_status_string(st)
        torch.cuda.synchronize()
        _, ref_out, ref_in = E.signed_distance(occ, 0.02, transform=E.edt_separable_minplus)
        got = d2.cpu().numpy().view(np.uint32).astype(np.int64)
        np.testing.assert_array_equal(got[0], ref_out)
        np.testing.assert_array_equal(got[1], ref_in)
