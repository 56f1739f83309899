"""AO and shadow grids built together under lights that are not unit vectors (any
finite vector but 0 is accepted and taken as it is): the samples' boxes in LDS are as
wide as the light is long."""
import numpy as np
import pytest

import oracle as O
import paper_1801_01155_amd as L
from paper_1801_01155_amd import synth

from . import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("light", [(0.0, 0.0, 1.9), (1.3, -1.6, 0.4), (0.2, 0.1, -0.3),
                                   (-3.0, 0.5, 2.0), (40.0, 1.0, -2.0)])
def test_shadow_of_long_lights(light):
    grid = (72, 64, 80)
    ls = synth.abc_lineset(3000, 120, 9, True)
    s = L.lineset_voxelize(ls.curve_off, grid, 32, xyz=ls.xyz, attr=ls.attr)
    L.lineset_build_lod(s, U.dev(synth.lut_importance_alpha()), opaque=False, build_ao=True,
                        build_shadow=True, light_dir=light)
    rho = L.lineset_export(s, L.EXPORT_LOD_RHO).cpu().numpy().astype(np.float64)
    sh = L.lineset_export(s, L.EXPORT_SHADOW).cpu().numpy()
    ao = L.lineset_export(s, L.EXPORT_AO).cpu().numpy()
    light = np.asarray(light, np.float32).astype(np.float64)
    # fp32: some ten samples of up to a dozen roundings each, the sum at most 1
    assert np.abs(sh - O.shadow_grid(rho, grid, light)).max() < 1e-5
    assert np.abs(ao - O.ao_grid(rho, grid)).max() < 1e-5
