"""Levels 0 and 1 of the density pyramid formed together, a wave per row of up to
64 voxels: rows around the limits (48 voxels: the kernel's shortest; 64 and 65:
one and two waves), single layers, odd sides, and lists far beyond one 64-record
step, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1801_01155_amd as L
from paper_1801_01155_amd import synth

from . import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(47, 5, 6), (48, 1, 1), (48, 5, 6), (64, 2, 2), (65, 7, 3),
                                  (129, 4, 9), (200, 1, 3)])
@pytest.mark.parametrize("n,opaque", [(3, False), (60, True), (4000, False)])
def test_rows(grid, n, opaque):
    rng = np.random.default_rng(n)
    lat = rng.integers(0, 256 * np.array(grid), size=(n, 4, 3)).astype(np.int32)
    if n > 1000:      # half of the curves in a corner: lists of hundreds
        lat[: n // 2] %= 700
        lat = np.minimum(lat, 256 * np.array(grid, np.int32) - 1)
    lat = lat.reshape(-1, 3)
    off = np.arange(n + 1, dtype=np.int64) * 4
    attr = (np.arange(n) * 37 % 256).astype(np.uint8)
    s = L.lineset_voxelize(off, grid, 32, lattice=lat, attr=attr)
    ref = O.voxelize(lat, off, attr, grid, 32)
    lut = synth.lut_importance_alpha()
    L.lineset_build_lod(s, U.dev(lut), opaque=opaque)
    torch.cuda.synchronize()
    cnt, ln, rho, dims, _ = O.lod(ref, grid, 32, lut, opaque=opaque)
    # fp32 sums of at most some hundred positive terms: 64 lanes by a tree, then
    # steps in turn; relative error below 1e-5 (each addition 6e-8)
    for what, r in ((L.EXPORT_LOD_COUNT, cnt), (L.EXPORT_LOD_LEN, ln), (L.EXPORT_LOD_RHO, rho)):
        g = L.lineset_export(s, what).cpu().numpy().astype(np.float64)
        assert np.allclose(g, r, rtol=1e-5, atol=1e-12)
    assert s.info().n_levels == len(dims)
