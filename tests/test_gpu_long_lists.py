"""Sets whose lists go by bricks and hold long voxels, which are listed apart (more
than 1024 lines, in bricks of more than 2048), some longer than a workgroup places
(8192): one or several in a brick, at the limits and far above them, in bricks whole
and cut, with and without per-vertex attributes, against the oracle bit for bit."""
import numpy as np
import pytest

import oracle as O
import paper_1801_01155_amd as L

from . import gpu_util as U
from .test_gpu_bricks import _long_segments

pytestmark = pytest.mark.gpu


def _bundle(voxel, m, seed):
    """m curves of one segment that enters a voxel and leaves it along x."""
    p = np.random.default_rng(seed).integers(0, 256, size=(m, 2, 3))
    p[:, 0, 0], p[:, 1, 0] = -100, 400
    return (p + 256 * np.asarray(voxel)).reshape(-1, 3).astype(np.int32)


@pytest.mark.parametrize("grid,curves,voxels,attrs", [
    ((128, 96, 112), 16000, [((40, 41, 42), 8192), ((42, 41, 42), 8193)], False),
    ((128, 96, 112), 16000, [((8, 17, 25), 9000), ((10, 16, 24), 9001), ((15, 23, 31), 30000)], True),
    ((130, 97, 113), 16000, [((128, 96, 112), 20000), ((1, 0, 0), 12000), ((64, 50, 51), 50000)], False),
    ((128, 96, 112), 2500, [((40, 41, 42), 1100), ((60, 41, 42), 1500), ((3, 70, 9), 1022),
                            ((3, 72, 9), 1026), ((100, 8, 90), 2100), ((101, 15, 92), 3000),
                            ((104, 8, 90), 8000), ((109, 9, 90), 900)], True)])
def test_long_voxels(grid, curves, voxels, attrs):
    a, off_a = _long_segments(grid, curves, 12, 3)
    parts, offs = [a], [off_a]
    for k, (v, m) in enumerate(voxels):
        # between the other curves, not behind them all
        parts.append(_bundle(v, m, k))
        offs.append(offs[-1][-1] + 2 * np.arange(1, m + 1))
        b, off_b = _long_segments(grid, curves // 40, 12, 10 + k)
        parts.append(b)
        offs.append(offs[-1][-1] + off_b[1:])
    lat, off = np.concatenate(parts), np.concatenate(offs)
    attr = (np.arange(len(off) - 1) % 251).astype(np.uint8)
    vattr = (np.arange(len(lat)) * 7 % 256).astype(np.uint8) if attrs else None
    s = L.lineset_voxelize(off, grid, 32, lattice=lat, attr=attr, vattr=vattr)
    ref = O.voxelize(lat, off, attr, grid, 32, vattr=vattr)
    n = np.diff(ref.offsets.astype(np.int64))
    # the brick path's range: at most 1/64 of the lines in one brick
    pad = np.pad(n.reshape(grid[::-1]), [(0, -g % 8) for g in grid[::-1]])
    z, y, x = (k // 8 for k in pad.shape)
    assert pad.reshape(z, 8, y, 8, x, 8).sum((1, 3, 5)).max() * 80 < n.sum()
    assert (n > 1024).any()
    offs, recs = U.gpu_csr(s)
    assert np.array_equal(offs, ref.offsets)
    assert np.array_equal(recs, ref.records)
    i = s.info()
    assert i.nonempty_voxels == int((n > 0).sum()) and i.max_list == int(n.max())
    if attrs:
        e = L.lineset_export(s, L.EXPORT_ENDS).cpu().numpy().view(np.uint16)
        assert np.array_equal(e, ref.ends)
