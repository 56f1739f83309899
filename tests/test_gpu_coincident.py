"""Lines whose two event points coincide, or nearly: curves that turn back on
plane crossings, edges and corners, with segment lengths that are powers of two
(2^16 x 2^16 x one lattice unit is a multiple of 2^32: the low halves of the
points' cross products agree although the points differ), against the oracle."""
import numpy as np
import pytest

import oracle as O
import paper_1801_01155_amd as L

from . import gpu_util as U

pytestmark = pytest.mark.gpu


def _curves(grid, n, length, seed):
    rng = np.random.default_rng(seed)
    top = 256 * np.array(grid, np.int64)
    p = rng.integers(0, top, size=(n, 3))
    p -= p % rng.choice([1, 2, 128, 256], size=(n, 1))
    out = [p]
    size = np.array([65536, 32768, 512, 256, 255, 1, 0])
    for _ in range(length - 1):
        s = rng.choice(size, size=(n, 3)) * rng.choice([-1, 1], size=(n, 3))
        # a third of the steps undo the one before (the same points again)
        if len(out) > 1:
            back = rng.random(n) < 0.34
            s[back] = (out[-2] - out[-1])[back] + rng.integers(-1, 2, size=(n, 3))[back]
        q = out[-1] + s
        q = np.where((q < 0) | (q >= top), out[-1] - s, q)
        q = np.where((q < 0) | (q >= top), out[-1], q)
        out.append(q)
    return np.stack(out, 1).reshape(-1, 3).astype(np.int32)


@pytest.mark.parametrize("grid", [(600, 530, 3), (3, 300, 300), (270, 4, 270)])
@pytest.mark.parametrize("seed,bins", [(1, 32), (2, 1), (3, 64)])
def test_coincident_points(grid, seed, bins):
    n, length = 700, 24
    lat = _curves(grid, n, length, seed)
    off = np.arange(n + 1, dtype=np.int64) * length
    vattr = (np.arange(len(lat)) * 11 % 256).astype(np.uint8)
    for va in (None, vattr):
        s = L.lineset_voxelize(off, grid, bins, lattice=lat, vattr=va)
        ref = O.voxelize(lat, off, None, grid, bins, vattr=va)
        offs, recs = U.gpu_csr(s)
        assert np.array_equal(offs, ref.offsets)
        assert np.array_equal(recs, ref.records)
