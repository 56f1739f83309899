"""The neighbour mode's sweeps (each list tested once as its voxel comes near, a
sorted buffer of hits ahead, a second sweep when it overflows) against the
oracle, at the sizes where they can go wrong: grids narrower than the
neighbourhood, lists far beyond the buffer and the queue, tubes almost a voxel
thick, and batched views, whose kernel forms the grown occupancy itself."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1801_01155_amd as L
from paper_1801_01155_amd import synth

from . import gpu_util as U

pytestmark = pytest.mark.gpu


def _lines(grid, n_curves, length, seed):
    rng = np.random.default_rng(seed)
    top = 256 * np.array(grid) - 1
    p = rng.integers(0, top + 1, size=(n_curves, 1, 3))
    q = np.clip(p + np.cumsum(rng.integers(-500, 501, size=(n_curves, length, 3)), axis=1), 0, top)
    off = np.arange(n_curves + 1, dtype=np.int64) * length
    return q.reshape(-1, 3).astype(np.int32), off


# (grid, curves, vertices, radius): lists average below one line per voxel, then
# tens (every neighbourhood overflows the 6-slot buffer), then hundreds (several
# queue fills per step)
@pytest.mark.parametrize("grid,n,length,radius", [
    ((1, 1, 1), 30, 12, 0.3), ((2, 1, 3), 40, 12, 0.4), ((5, 2, 9), 60, 10, 0.4),
    ((37, 18, 26), 25, 20, 0.4), ((37, 18, 26), 25, 20, 0.97), ((8, 7, 6), 700, 12, 0.05),
    ((4, 4, 4), 1500, 12, 0.02), ((64, 4, 5), 120, 30, 0.6)])
@pytest.mark.parametrize("opaque", [False, True])
def test_neighbour_sweeps(grid, n, length, radius, opaque):
    lat, off = _lines(grid, n, length, 3 * n + sum(grid))
    s = L.lineset_voxelize(off, grid, 16, lattice=lat)
    ref = O.voxelize(lat, off, None, grid, 16)
    lut = synth.lut_ramp(1.0) if opaque else synth.lut_constant(alpha=0.05)
    cams = [synth.orbit_cameras(grid, 1, 5, 40, 24)[0],
            synth.orbit_cameras(grid, 1, 6, 24, 40, True)[0],
            # along an axis, rays on lattice planes and half-way between
            synth.Camera((-3.0, 0.5 * grid[1], 0.5 * grid[2]), (1, 0, 0),
                         (0, 0.5 * grid[1], 0), (0, 0, 0.5 * grid[2]), 32, 32, True)]
    # transparent rays never end early (alpha_stop 2), opaque ones at their
    # first fragment (the oracle counts on past it with alpha_stop above 1)
    kw = dict(radius=radius, mode=1, opaque=opaque, shading=1,
              alpha_stop=0.95 if opaque else 2.0, merge_curves=False)
    good = total = 0
    for cam in cams:
        g, kg = L.lineset_render_counted(s, cam, U.dev(lut), **kw)
        r, cnt = O.render(ref, grid, 16, cam, lut=lut, **kw)
        torch.cuda.synchronize()
        # the counts differ only by fp32 / fp64 silhouette flips
        assert abs(kg["fragments"] - cnt["fragments"]) <= 2 + 2e-3 * cnt["fragments"]
        d = np.abs(g.cpu().numpy() - r).max(axis=-1)
        good += int((d <= U.IMAGE_TOL).sum())
        total += d.size
        # the batched kernel (no grown occupancy handed over): bit for bit
        out = torch.empty_like(g)
        b = L.Batch([(s, cam, U.dev(lut), out, kw)])
        b.render()
        torch.cuda.synchronize()
        b.close()
        assert torch.equal(out, g)
    # thin tubes over hundreds of lines: a silhouette flip is one of many
    # layers of opacity 0.05, so it stays rare but not below one in a thousand
    # of these small images; one pixel in a hundred bounds it
    assert good >= 0.99 * total, (good, total)
