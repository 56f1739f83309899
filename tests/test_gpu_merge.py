"""The merge passes of lineset_update on lists that begin, end and run on across
their 64-record chunks and 64-voxel waves, against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle as O
import paper_1801_01155_amd as L

from . import gpu_util as U

pytestmark = pytest.mark.gpu


def _curves(grid, n, length, seed):
    rng = np.random.default_rng(seed)
    top = 256 * np.array(grid)
    return rng.integers(0, top, size=(n, length, 3)).astype(np.int32)


# lists of hundreds (one voxel over many chunks), of about 64, of a few, and
# mostly empty ones; the last wave of voxels is partial in all but the first
@pytest.mark.parametrize("grid,n", [((4, 4, 4), 1500), ((9, 5, 7), 2000), ((33, 10, 21), 400),
                                    ((70, 61, 35), 60)])
@pytest.mark.parametrize("remove,add", [(0.4, 30), (1.0, 0), (0.0, 25), (1.0, 40), (0.01, 1)])
def test_merge(grid, n, remove, add):
    old, new = _curves(grid, n, 6, n), _curves(grid, max(add, 1), 6, n + 1)[:add]
    rng = np.random.default_rng(add)
    gone = np.flatnonzero(rng.random(n) < remove)
    off = lambda m: np.arange(m + 1, dtype=np.int64) * 6  # noqa: E731
    attr, nattr = (np.arange(n) % 256).astype(np.uint8), (np.arange(add) % 256).astype(np.uint8)
    s = L.lineset_voxelize(off(n), grid, 16, lattice=old.reshape(-1, 3), attr=attr)
    kw = dict(curve_off=off(add), lattice=new.reshape(-1, 3), attr=nattr) if add else {}
    L.lineset_update(s, remove=gone if len(gone) else None, **kw)
    # a removed curve keeps its id and has no vertices
    keep = np.ones(n + add, bool)
    keep[gone] = False
    ref_off = np.concatenate([[0], np.cumsum(6 * keep)]).astype(np.int64)
    lat = np.concatenate([old, new])[keep].reshape(-1, 3)
    ref = O.voxelize(lat, ref_off, np.concatenate([attr, nattr]), grid, 16)
    offs, recs = U.gpu_csr(s)
    assert np.array_equal(offs, ref.offsets)
    assert np.array_equal(recs, ref.records)
    i = s.info()
    m = np.diff(ref.offsets.astype(np.int64))
    assert i.nonempty_voxels == int((m > 0).sum()) and i.max_list == int(m.max())
