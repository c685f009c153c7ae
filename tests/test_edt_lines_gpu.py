"""The y and z passes of the distance field at the sizes where their work split changes:
lines of 64 / 65, 256 / 257, 384 / 385 and 512 samples (8, 16 or 32 outputs per unit, 8- or
16-bit row indices), whole and partial units of 8 outputs, and line counts around the
32 lines of a block.  Every result is an integer, so the bound is equality."""
import numpy as np
import pytest

from oracle import edt as E
from tests.test_edt_gpu import check

pytestmark = pytest.mark.gpu


def _scenes(n_z, n_y, n_x, axis, seed):
    """Sparse sources, their complement, and slabs that fill or empty whole lines."""
    rng = np.random.default_rng(seed)
    sparse = rng.uniform(size=(n_z, n_y, n_x)) < 0.01
    slab = np.zeros_like(sparse)
    n = sparse.shape[axis]
    at = [slice(None)] * 3
    at[axis] = slice(n // 4, n // 4 + max(1, n // 3))
    slab[tuple(at)] = True          # thick obstacle, free on both sides
    slab[:, :, 0] = False           # a line with no obstacle
    slab[:, :, n_x - 1] = True      # a line with no free voxel
    return sparse, ~sparse, slab


@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 64, 65, 127, 128, 129, 255, 256, 257, 383, 384, 385, 511,
                               512])
@pytest.mark.parametrize("axis", [0, 1])
def test_line_lengths(n, axis):
    other, n_x = (3, 11) if n % 2 else (2, 16)   # 33 lines, or 32
    shape = (n, other, n_x) if axis == 0 else (other, n, n_x)
    for occ in _scenes(*shape, axis, n + axis):
        check(occ, 0.01, transform=E.edt_separable_minplus)
