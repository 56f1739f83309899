"""Sets on either side of the rule that sends lists by bricks or by rank atomics: few
and many lines, dense and sparse grids, lines crowded into few bricks. Lists, list
statistics and occupancy-dependent images are those of the oracle, bit for bit."""
import numpy as np
import pytest

import oracle as O
import paper_1801_01155_amd as L

from . import gpu_util as U
from .test_gpu_bricks import _long_segments

pytestmark = pytest.mark.gpu


def _check(lat, off, grid, lo, hi):
    attr = (np.arange(len(off) - 1) % 251).astype(np.uint8)
    s = L.lineset_voxelize(off, grid, 32, lattice=lat, attr=attr)
    i = s.info()
    assert lo <= i.n_record_slots <= hi, i.n_record_slots   # the side of the rule meant
    ref = O.voxelize(lat, off, attr, grid, 32)
    offs, recs = U.gpu_csr(s)
    assert np.array_equal(offs, ref.offsets)
    assert np.array_equal(recs, ref.records)
    n = np.diff(ref.offsets.astype(np.int64))
    assert i.nonempty_voxels == int((n > 0).sum()) and i.max_list == int(n.max())


M = 1 << 20


@pytest.mark.parametrize("grid,lines,lo,hi", [
    ((128, 128, 64), 0.8e6, 0, M - 1),            # too few lines for bricks
    ((128, 128, 64), 1.6e6, M, 3 * M),
    ((128, 128, 64), 7e6, 5 * M, 10 * M),         # more than 2048 lines per brick on average
    ((256, 200, 160), 1.4e6, M, 2 * M),           # 16640 bricks: about 80 each
    ((300, 280, 310), 1.6e6, M, 2 * M),           # 57600 bricks: below 48 each
    ((1024, 1024, 1), 2.2e6, M, 4 * M)])
def test_even_sets(grid, lines, lo, hi):
    n_curves = int(lines / (9 * sum(grid) / 3))
    lat, off = _long_segments(grid, n_curves, 10, sum(grid))
    _check(lat, off, grid, lo, hi)


@pytest.mark.parametrize("side", [12, 24, 48, 80])
def test_crowded_sets(side):
    # all lines in side^3 voxels of 160^3 but for a few curves across the grid
    grid = (160, 160, 160)
    lo = np.array([32, 40, 24])
    a, off_a = _long_segments(grid, 50, 4, 5)
    n_curves = int(2e6 / (9 * side))
    b, off_b = _long_segments(grid, n_curves, 10, side, (256 * lo, 256 * (lo + side)))
    lat, off = np.concatenate([a, b]), np.concatenate([off_a, off_a[-1] + off_b[1:]])
    _check(lat, off, grid, M, 4 * M)


def test_vertices_that_give_no_segment():
    # curves of one and two vertices: half the sampled pairs belong to no curve
    grid = (128, 128, 64)
    a, off_a = _long_segments(grid, 60000, 2, 8)
    one = np.random.default_rng(9).integers(0, 256 * 64, size=(5000, 3)).astype(np.int32)
    lat = np.concatenate([a, one])
    off = np.concatenate([off_a, off_a[-1] + 1 + np.arange(len(one))])
    _check(lat, off, grid, M, 8 * M)
