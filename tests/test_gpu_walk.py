"""The ray caster's grid walk: coarse steps over empty macro cells against the
oracle's fine stepping, on rays whose plane crossings coincide."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1801_01155_amd as L
from paper_1801_01155_amd import synth

from . import gpu_util as U

pytestmark = pytest.mark.gpu


def _sparse(grid, seed, n_curves=14):
    """A few random polylines: most macro cells stay empty."""
    rng = np.random.default_rng(seed)
    top = 256 * np.array(grid) - 1
    lat, off = [], [0]
    for _ in range(n_curves):
        p = rng.integers(0, top + 1)
        n = int(rng.integers(2, 9))
        q = p + np.cumsum(rng.integers(-700, 701, size=(n, 3)), axis=0)
        lat.append(np.clip(q, 0, top))
        off.append(off[-1] + n)
    return np.concatenate(lat).astype(np.int32), np.array(off, np.int64)


def _tie_cameras(grid):
    """Parallel rays along axes and diagonals, both ways, starting on lattice
    points and half-way between them: crossings of several planes coincide."""
    g = np.array(grid, np.float64)
    cams = []
    for f, r, u in (((1, 0, 0), (0, 1, 0), (0, 0, 1)), ((0, -1, 0), (1, 0, 0), (0, 0, 1)),
                    ((1, 1, 0), (1, -1, 0), (0, 0, 1)), ((-1, 1, 1), (1, 1, 0), (1, 0, 1)),
                    ((1, 1, 1), (1, -1, 0), (1, 0, -1)), ((-2, -1, 4), (0, 4, 1), (2, 0, 1))):
        f, r, u = (np.array(x, np.float64) for x in (f, r, u))
        eye = np.floor(g / 2) - 64 * f
        s = float(max(grid) // 2 + 2) / 2
        cams.append(synth.Camera(tuple(eye), tuple(f), tuple(s * r), tuple(s * u), 24, 16, True))
    return cams


@pytest.mark.parametrize("grid", [(1, 1, 1), (4, 4, 4), (5, 3, 9), (33, 18, 7), (40, 41, 43),
                                  (64, 5, 31)])
def test_coarse_walk_meets_the_same_voxels(grid):
    lat, off = _sparse(grid, 7 + sum(grid))
    s = L.lineset_voxelize(off, grid, 16, lattice=lat)
    ref = O.voxelize(lat, off, None, grid, 16)
    lut = synth.lut_constant(alpha=0.01)
    cams = _tie_cameras(grid)
    cams += synth.orbit_cameras(grid, 4, 3, 24, 16) + synth.orbit_cameras(grid, 2, 4, 24, 16, True)
    for k, cam in enumerate(cams):
        kw = dict(radius=0.4, opaque=False, alpha_stop=2.0, merge_curves=False, shading=0)
        g, kg = L.lineset_render_counted(s, cam, U.dev(lut), **kw)
        r, cnt = O.render(ref, grid, 16, cam, lut=lut, **kw)
        # the rays never stop early: every voxel and line of every ray is counted
        assert kg["nonempty"] == cnt["nonempty"], (grid, k)
        assert kg["tested"] == cnt["tested"], (grid, k)
        assert kg["visited"] <= cnt["visited"]
        torch.cuda.synchronize()
        # shading off: a pixel differs only where a silhouette test flips (one
        # layer, 0.01); at most one pixel in a hundred of these small images
        d = np.abs(g.cpu().numpy() - r).max(axis=-1)
        assert (d > 1e-4).mean() <= 0.01, (grid, k)


# image sizes (8 x 8 pixel tiles) around the limits of every split: one ray per
# workgroup, 32, 16, 8, 4 ways, and whole tiles; ragged edges
@pytest.mark.parametrize("w,h", [(1, 1), (7, 9), (130, 97), (201, 160), (322, 257), (450, 401),
                                 (641, 480)])
@pytest.mark.parametrize("opaque,mode", [(True, 0), (False, 0), (True, 1), (False, 1)])
def test_split_tiles_give_the_whole_image(w, h, opaque, mode):
    ls = synth.abc_lineset(400, 60, 9)
    grid = (48, 40, 56)
    s = L.lineset_voxelize(ls.curve_off, grid, 32, xyz=ls.xyz, attr=ls.attr)
    lut = U.dev(synth.lut_ramp(1.0) if opaque else synth.lut_importance_alpha())
    cam = synth.orbit_cameras(grid, 1, w, w, h, orthographic=bool(w & 1))[0]
    kw = dict(radius=0.4, mode=mode, opaque=opaque, shading=1)
    out = torch.empty((h, w, 4), dtype=torch.float32, device="cuda")
    b = L.Batch([(s, cam, lut, out, kw)])       # renders whole tiles
    b.render()
    for _ in range(3):                          # first and repeated frames of the view
        img = torch.full((h, w, 4), -1.0, device="cuda")
        L.lineset_render(s, cam, lut, out=img, **kw)
        assert torch.equal(img, out)
    b.close()
