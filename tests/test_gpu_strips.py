"""Images much longer than wide and views off the image's centre: the launch covers
the image's tiles, however far the rings around the grid's centre would reach."""
import numpy as np
import pytest
import torch

import paper_1801_01155_amd as L
from paper_1801_01155_amd import synth

from . import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lines():
    ls = synth.abc_lineset(400, 60, 9)
    grid = (48, 40, 56)
    return grid, L.lineset_voxelize(ls.curve_off, grid, 32, xyz=ls.xyz, attr=ls.attr)


def _camera(grid, w, h, shift, ortho):
    """The grid fills the image; its centre lies `shift` half images to the left and half
    as far below (1: at the left edge)."""
    c = synth.look_camera(grid, w, h, (0.3, -1.0, 0.4), ortho)
    f, u = np.array(c.forward), np.array(c.up)
    r = np.array(c.right) * (np.linalg.norm(u) / np.linalg.norm(c.right))
    if ortho:
        return synth.Camera(tuple(np.array(c.eye) + shift * (r + 0.5 * u)), c.forward, tuple(r), c.up,
                            w, h, True)
    return synth.Camera(c.eye, tuple(f + shift * (r + 0.5 * u)), tuple(r), c.up, w, h, False)


def _check(lines, w, h, opaque, mode, shift, ortho):
    grid, s = lines
    lut = U.dev(synth.lut_ramp(1.0) if opaque else synth.lut_importance_alpha())
    cam = _camera(grid, w, h, shift, ortho)
    kw = dict(radius=0.4, mode=mode, opaque=opaque, shading=1)
    out = torch.empty((h, w, 4), dtype=torch.float32, device="cuda")
    b = L.Batch([(s, cam, lut, out, kw)])       # renders whole tiles
    b.render()
    torch.cuda.synchronize()
    assert float(out[..., 3].max()) > 0.0       # the grid is in the image
    for _ in range(3):                          # first and repeated frames of the view
        img = torch.full((h, w, 4), -1.0, device="cuda")
        L.lineset_render(s, cam, lut, out=img, **kw)
        assert torch.equal(img, out)
    b.close()


# transparent neighbour-mode frames are ordered by tile times; their split rings
# hold up to 4000 times the image's tiles
@pytest.mark.parametrize("w,h", [(4096, 8), (2048, 61), (16384, 5), (256, 256)])
@pytest.mark.parametrize("shift,ortho", [(0.0, True), (1.0, True), (1.0, False)])
def test_ordered_strips(lines, w, h, shift, ortho):
    _check(lines, w, h, False, 1, shift, ortho)


# small frames split all their tiles; longer strips are whole or ordered
@pytest.mark.parametrize("w,h", [(4096, 8), (8, 4096), (2048, 61), (32768, 8), (16384, 5),
                                 (256, 256), (401, 300)])
@pytest.mark.parametrize("opaque,mode", [(True, 0), (False, 0), (True, 1)])
@pytest.mark.parametrize("shift,ortho", [(0.0, True), (1.0, True), (1.0, False)])
def test_strips_and_edges(lines, w, h, opaque, mode, shift, ortho):
    _check(lines, w, h, opaque, mode, shift, ortho)
