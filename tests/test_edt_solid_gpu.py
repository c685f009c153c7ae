"""Distance fields of solid grids: leaves whose D_in search could go beyond its reach (64 rows,
judged after 8) leave D_in to the scan between cuts that gives D_out.  Values by equality at
the thicknesses and line lengths where that changes; and the time of a solid grid, which may
not grow with the thickness: the search of a leaf ends after 8 rows or goes on for 64 (about
the work of one scan), then one scan gives D_in and one D_out, so a grid takes at most
three times what its complement, one scan, takes."""
import numpy as np
import pytest

from oracle import edt as E
from tests.test_edt_gpu import check

pytestmark = pytest.mark.gpu


def _scenes(n, axis, seed):
    """Lines of n voxels along `axis` (0: z, 1: y) over rows of 150."""
    rng = np.random.default_rng(seed)
    shape = (n, 2, 150) if axis == 0 else (2, n, 150)

    def rows(mask):   # occupied where mask[p] holds for the line's p-th plane (or row)
        return np.broadcast_to(mask.reshape((n, 1, 1) if axis == 0 else (1, n, 1)), shape).copy()

    for thick in (8, 15, 16, 17, 24, 25, 26, 33, 126, 129, 136, 137, 145):
        mask, at = np.zeros(n, bool), int(rng.integers(0, 9))
        while at < n:
            mask[at:at + thick] = True
            at += thick + int(rng.integers(1, 20))
        yield rows(mask)                            # slabs: no free voxel in their planes
    solid = rng.uniform(size=shape) >= 0.0004
    yield solid                                     # few free voxels, samples of all sizes
    yield ~solid
    solid[..., :40] = rng.uniform(size=shape)[..., :40] < 0.5
    yield solid                                     # beside thin ones, in one block too
    solid[..., 60:70] = False
    yield solid                                     # lines without an obstacle in it
    one = np.ones(shape, bool)
    one[0, 0, 149] = False
    yield one
    yield np.ones(shape, bool)


@pytest.mark.parametrize("n", [8, 9, 16, 17, 33, 64, 65, 128, 129, 200, 256, 257, 384, 385, 512])
@pytest.mark.parametrize("axis", [0, 1])
def test_solid_lines(n, axis):
    for occ in _scenes(n, axis, 2 * n + axis):
        check(occ, 0.01, transform=E.edt_separable_minplus)


def _us(occ):
    import torch

    from paper_2512_22575_amd import smpc as S
    nz, ny, nx = occ.shape
    need = S.smpc_edt_workspace_bytes(nx, ny, nz)
    d = torch.from_numpy(occ.astype(np.uint8)).cuda()
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    phi = torch.empty(occ.shape, device="cuda")
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    times = []
    for _ in range(7):
        a.record()
        for _ in range(20):
            st = S.smpc_edt(d.data_ptr(), nx, ny, nz, 0.02, phi.data_ptr(), None, work.data_ptr(),
                            need, torch.cuda.current_stream().cuda_stream)
            assert st == S.SMPC_OK
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / 20)
    return float(np.median(times))


@pytest.mark.parametrize("what", ["full", "one free voxel", "floor layer"])
def test_time_of_solid_grids(what):
    occ = np.zeros((64, 512, 200) if what == "floor layer" else (300, 300, 100), bool)
    if what == "floor layer":
        occ[0] = True
        other = np.zeros_like(occ)
    else:
        occ[:] = True
        if what == "one free voxel":
            occ[150, 150, 50] = False
        other = ~occ
    t, ref = _us(occ), _us(other)
    print(f"{what}: {t:.1f} us, reference {ref:.1f} us", flush=True)
    assert t <= 3.0 * ref
