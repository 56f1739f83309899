"""Occupancy words and list statistics at the edges of their launches: cells per
workgroup, the two splits of a cell, sides that are no multiple of 4, against
the lists themselves; the rays' counts of non-empty voxels need every bit."""
import numpy as np
import pytest

import oracle as O
import paper_1801_01155_amd as L
from paper_1801_01155_amd import synth

from . import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(1, 1, 1), (5, 3, 2), (4, 4, 260), (7, 66, 9), (80, 80, 81),
                                  (128, 64, 64), (128, 64, 65), (127, 64, 68), (130, 66, 66)])
@pytest.mark.parametrize("n_curves", [1, 40, 3000])
def test_statistics_and_counts(grid, n_curves):
    rng = np.random.default_rng(n_curves)
    top = 256 * np.array(grid)
    lat = rng.integers(0, top, size=(n_curves, 4, 3))
    lat[:, 1:] = np.clip(lat[:, :1] + rng.integers(-600, 601, size=(n_curves, 3, 3)), 0, top - 1)
    lat = lat.reshape(-1, 3).astype(np.int32)
    off = np.arange(n_curves + 1, dtype=np.int64) * 4
    s = L.lineset_voxelize(off, grid, 32, lattice=lat)
    ref = O.voxelize(lat, off, None, grid, 32)
    n = np.diff(ref.offsets.astype(np.int64))
    i = s.info()
    assert i.nonempty_voxels == int((n > 0).sum())
    assert i.max_list == int(n.max())
    lut = synth.lut_constant(alpha=0.01)
    kw = dict(radius=0.4, opaque=False, alpha_stop=2.0, merge_curves=False, shading=0)
    for cam in synth.orbit_cameras(grid, 2, 3, 40, 32):
        _, kg = L.lineset_render_counted(s, cam, U.dev(lut), **kw)
        _, cnt = O.render(ref, grid, 32, cam, lut=lut, **kw)
        assert kg["nonempty"] == cnt["nonempty"]
