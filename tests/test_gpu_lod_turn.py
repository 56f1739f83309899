"""Levels 0 and 1 of the density pyramid over grids of one to nine blocks to a row,
with enough rows that the columns of blocks turn, and on either side of the rule
that forms the two levels together (sides, idle lanes, voxels), against the oracle."""
import numpy as np
import pytest

import oracle as O
import paper_1801_01155_amd as L
from paper_1801_01155_amd import synth

from . import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(31, 9, 9), (32, 9, 9), (95, 40, 33), (96, 40, 33), (128, 70, 66),
                                  (190, 90, 50), (250, 131, 60), (330, 41, 30), (512, 80, 20),
                                  (520, 60, 22), (213, 250, 236), (214, 250, 236)])
def test_turned_rows(grid):
    ls = synth.abc_lineset(800, 60, sum(grid), False)
    # the flow spread over the whole grid, whatever its sides
    lo, hi = ls.xyz.min(0), ls.xyz.max(0)
    lat = ((ls.xyz - lo) / (hi - lo) * (256 * np.array(grid) - 1)).astype(np.int32)
    s = L.lineset_voxelize(ls.curve_off, grid, 32, lattice=lat, attr=ls.attr)
    ref = O.voxelize(lat, ls.curve_off, ls.attr, grid, 32)
    lut = synth.lut_importance_alpha()
    L.lineset_build_lod(s, U.dev(lut), opaque=False)
    cnt, ln, rho, _, _ = O.lod(ref, grid, 32, lut, opaque=False)
    # fp32 sums of at most some hundred positive terms (each addition 6e-8)
    for what, r in ((L.EXPORT_LOD_COUNT, cnt), (L.EXPORT_LOD_LEN, ln), (L.EXPORT_LOD_RHO, rho)):
        g = L.lineset_export(s, what).cpu().numpy().astype(np.float64)
        assert np.allclose(g, r, rtol=1e-5, atol=1e-12)
