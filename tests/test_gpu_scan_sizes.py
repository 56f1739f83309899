"""Prefix sums at the sizes where their launches change (one tile of 4096, up to
1024 tiles, more): voxel counts of the grid and curve counts, against the
oracle, bit for bit."""
import numpy as np
import pytest

import oracle as O
import paper_1801_01155_amd as L

from . import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(1, 1, 1), (16, 16, 16), (17, 241, 1), (64, 64, 2),
                                  (128, 128, 256), (128, 128, 257)])
@pytest.mark.parametrize("n_curves", [1, 4095, 4096, 4097, 9000])
def test_sizes(grid, n_curves):
    rng = np.random.default_rng(n_curves)
    lat = rng.integers(0, 256 * np.array(grid), size=(n_curves, 3, 3))
    lat[:, 1:] = np.clip(lat[:, :1] + rng.integers(-400, 401, size=(n_curves, 2, 3)), 0,
                         256 * np.array(grid) - 1)
    lat = lat.reshape(-1, 3).astype(np.int32)
    off = np.arange(n_curves + 1, dtype=np.int64) * 3
    s = L.lineset_voxelize(off, grid, 32, lattice=lat)
    ref = O.voxelize(lat, off, None, grid, 32)
    offs, recs = U.gpu_csr(s)
    assert np.array_equal(offs, ref.offsets)
    assert np.array_equal(recs, ref.records)
    i = s.info()
    n = np.diff(ref.offsets.astype(np.int64))
    assert i.nonempty_voxels == int((n > 0).sum()) and i.max_list == int(n.max())
