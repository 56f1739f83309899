"""Prefix sums of large tiles (16384 items) at the sizes where their launches
change (up to 1024 of them, more) and with remainders, against the oracle, bit for bit.
"""
import numpy as np
import pytest

import oracle as O
import paper_1801_01155_amd as L

from . import gpu_util as U

pytestmark = pytest.mark.gpu


def _lattice(grid, n_curves, seed):
    rng = np.random.default_rng(seed)
    top = 256 * np.array(grid)
    lat = rng.integers(0, top, size=(n_curves, 3, 3))
    lat[:, 1:] = np.clip(lat[:, :1] + rng.integers(-900, 901, size=(n_curves, 2, 3)), 0, top - 1)
    return lat.reshape(-1, 3).astype(np.int32)


@pytest.mark.parametrize("grid", [(256, 256, 65), (1, 1023, 1024), (256, 256, 256),
                                  (255, 257, 256), (256, 256, 257)])
def test_large_tiles(grid):
    n_curves = 20000
    lat = _lattice(grid, n_curves, grid[1])
    off = np.arange(n_curves + 1, dtype=np.int64) * 3
    s = L.lineset_voxelize(off, grid, 32, lattice=lat)
    ref = O.voxelize(lat, off, None, grid, 32)
    offs, recs = U.gpu_csr(s)
    assert np.array_equal(offs, ref.offsets)
    assert np.array_equal(recs, ref.records)
