"""Voxelization by bricks (grids from 2^20 voxels, sets from 2^22 lines) against
the oracle, bit for bit: ragged brick blocks, bricks of more lines than one
workgroup places at once, voxels longer than its LDS, per-vertex attributes."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1801_01155_amd as L

from . import gpu_util as U

pytestmark = pytest.mark.gpu


def _long_segments(grid, n_curves, n_vertices, seed, box=None):
    """Polylines whose segments cross many voxels; every third curve runs on
    lattice diagonals through voxel corners (several planes in one event)."""
    rng = np.random.default_rng(seed)
    lo, hi = (np.zeros(3, np.int64), 256 * np.array(grid)) if box is None else box
    p = rng.integers(lo, hi, size=(n_curves, n_vertices, 3))
    m = n_curves // 3
    d = rng.integers(1, max(2, int((hi - lo).min()) // 256), size=(m, 1, 1))
    s = rng.choice([-1, 1], size=(m, n_vertices, 3))
    p[:m] = np.clip((p[:m, :1] // 256) * 256 + 256 * d * s, lo, hi - 1)
    off = np.arange(n_curves + 1, dtype=np.int64) * n_vertices
    return p.reshape(-1, 3).astype(np.int32), off


def _check(lat, off, grid, bins, vattr=None):
    attr = (np.arange(len(off) - 1) % 251).astype(np.uint8)
    s = L.lineset_voxelize(off, grid, bins, lattice=lat, attr=attr, vattr=vattr)
    i = s.info()
    assert i.n_record_slots >= 1 << 22          # the brick path's range
    ref = O.voxelize(lat, off, attr, grid, bins, vattr=vattr)
    offs, recs = U.gpu_csr(s)
    assert np.array_equal(offs, ref.offsets)
    assert np.array_equal(recs, ref.records)
    n = np.diff(ref.offsets.astype(np.int64))
    assert i.nonempty_voxels == int((n > 0).sum()) and i.max_list == int(n.max())
    if vattr is not None:
        e = L.lineset_export(s, L.EXPORT_ENDS).cpu().numpy().view(np.uint16)
        assert np.array_equal(e, ref.ends)
    return n.reshape(grid[2], grid[1], grid[0])


def _brick_lines(n):
    pad = [(0, -s % 8) for s in n.shape]
    z, y, x = (s // 8 for s in np.pad(n, pad).shape)
    return np.pad(n, pad).reshape(z, 8, y, 8, x, 8).sum((1, 3, 5))


@pytest.mark.parametrize("grid,bins,attrs", [((128, 128, 64), 32, False),
                                             ((241, 107, 83), 16, True), ((97, 33, 340), 8, False)])
def test_bricks_on_ragged_grids(grid, bins, attrs):
    n_curves = int(8e6 / (9 * sum(grid) / 3))
    lat, off = _long_segments(grid, n_curves, 10, sum(grid))
    vattr = (np.arange(len(lat)) * 7 % 256).astype(np.uint8) if attrs else None
    _check(lat, off, grid, bins, vattr)


def test_bricks_beyond_a_workgroup():
    # a third of the lines in 5 x 3 x 3 bricks: one to many voxel ranges each
    grid = (128, 96, 112)
    a, off_a = _long_segments(grid, 6000, 12, 1)
    b, off_b = _long_segments(grid, 16000, 12, 2,
                              (256 * np.array([40, 16, 24]), 256 * np.array([80, 40, 48])))
    lat, off = np.concatenate([a, b]), np.concatenate([off_a, off_a[-1] + off_b[1:]])
    lines = _brick_lines(_check(lat, off, grid, 32))
    assert lines.max() > 3 * 8192 and ((lines > 2048) & (lines <= 8192)).any()


def test_voxel_longer_than_a_workgroup():
    # 9000 curves cross one voxel (its list leaves the brick path), beside others
    grid = (128, 96, 112)
    a, off_a = _long_segments(grid, 8000, 12, 3)
    rng = np.random.default_rng(4)
    m = 9000
    b = np.empty((m, 2, 3), np.int64)
    b[:, :, 1:] = 256 * 50 + rng.integers(0, 256, size=(m, 2, 2))
    b[:, 0, 0], b[:, 1, 0] = 256 * 59 + 9, 256 * 62 + 9
    lat = np.concatenate([a, b.reshape(-1, 3).astype(np.int32)])
    off = np.concatenate([off_a, off_a[-1] + 2 * np.arange(1, m + 1)])
    n = _check(lat, off, grid, 32)
    assert n.max() > 8192
