"""AO of the column kernel against its definition in 64 bits: as close as trilinear
samples are in fp32 whose weights come from 64-bit coordinates and are rounded once
(interpolations by differences along x, y, z), evaluated here step by step. The
kernel goes by four products per plane instead; on random cells their roundings come
to 4 % more at most."""
import math

import pytest
import torch

import oracle as O
import paper_1801_01155_amd as L
from paper_1801_01155_amd import synth

from . import gpu_util as U

pytestmark = pytest.mark.gpu


def _f32(x):
    return x.float().double()


def _lerp(w, a, b, fp32):
    # fp32: a rounded difference, then one fused multiply-add
    return _f32(w * _f32(b - a) + a) if fp32 else a + w * (b - a)


def _cone(levels, grid, u, s_max, fp32):
    rnd = _f32 if fp32 else (lambda x: x)
    v = torch.meshgrid(*[torch.arange(n, device="cuda") for n in grid[::-1]], indexing="ij")[::-1]
    occ = torch.zeros(v[0].shape, dtype=torch.float64, device="cuda")
    inside = torch.ones_like(occ, dtype=torch.bool)
    s = 1.0
    while s < s_max:
        for a in range(3):
            x = (v[a].double() + 0.5) + s * u[a]
            inside &= (x >= 0) & (x < grid[a])
        if not bool(inside.any()):
            break
        D = max(1.0, s)
        lv = min(len(levels) - 1, int(math.log2(D)))
        lev = levels[lv]
        lo, hi, fr = [], [], []
        for a in range(3):
            t = ((v[a] % 2 ** lv).double() + (0.5 + s * u[a])) / 2.0 ** lv - 0.5
            i = torch.floor(t)
            c, n = (v[a] >> lv) + i.long(), lev.shape[2 - a]
            lo.append(c.clamp(0, n - 1))
            hi.append((c + 1).clamp(0, n - 1))
            fr.append(rnd(t - i))
        tap = lambda k: lev[(hi if k & 4 else lo)[2], (hi if k & 2 else lo)[1],  # noqa: E731
                            (hi if k & 1 else lo)[0]]
        c = [_lerp(fr[0], tap(2 * k), tap(2 * k + 1), fp32) for k in range(4)]
        p = [_lerp(fr[1], c[2 * k], c[2 * k + 1], fp32) for k in range(2)]
        occ = torch.where(inside & (occ < 1.0), rnd(_lerp(fr[2], p[0], p[1], fp32) * D + occ), occ)
        s += D
    return occ.clamp(max=1.0)


@pytest.mark.parametrize("grid,cones,radius", [
    ((96, 96, 96), 16, 15.0), ((121, 70, 99), 8, 7.0), ((96, 96, 96), 3, 15.0)])
def test_error_against_64_bits(grid, cones, radius):
    ls = synth.abc_lineset(6000, 120, 17, True)
    s = L.lineset_voxelize(ls.curve_off, grid, 32, xyz=ls.xyz, attr=ls.attr)
    L.lineset_build_lod(s, U.dev(synth.lut_importance_alpha()), opaque=False, build_ao=True,
                        ao_cones=cones, ao_radius=radius, build_shadow=True,
                        light_dir=synth.LIGHT_DIR)
    rho = L.lineset_export(s, L.EXPORT_LOD_RHO).double()
    levels, d, at = [], list(grid), 0
    while at < rho.numel():
        n = d[0] * d[1] * d[2]
        levels.append(rho[at:at + n].reshape(d[2], d[1], d[0]))
        at, d = at + n, [(k + 1) // 2 for k in d]
    ao = {}
    for fp32 in (False, True):
        rnd = _f32 if fp32 else (lambda x: x)
        total = 0.0
        for u in O.fibonacci_dirs(cones):
            total = rnd(total + _cone(levels, grid, [float(c) for c in u], radius, fp32))
        ao[fp32] = rnd(1.0 - rnd(total / cones))
    got = L.lineset_export(s, L.EXPORT_AO).double().reshape(grid[::-1])
    rms = lambda x: float((x - ao[False]).square().mean().sqrt())  # noqa: E731
    print(f"[cone error {grid} {cones}] kernel={rms(got):.4e} fp32={rms(ao[True]):.4e}", flush=True)
    assert rms(got) <= 1.04 * rms(ao[True])
