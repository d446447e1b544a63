"""Voxel-driven backprojector: detector footprints in LDS and the views that
are sampled from memory instead, at every column length, against the FP64
oracle (relative L2 <= 1e-5: FP32 blends of positions within 1e-6 pixel).
"""

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_30166_amd import CylinderGeometry, Geometry

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _rel(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b)


def _roll(P, deg):
    """Turn the detector in its plane: u then varies along z."""
    a = np.radians(deg)
    R = np.array([[np.cos(a), -np.sin(a), 3.0], [np.sin(a), np.cos(a), -2.0], [0, 0, 1.0]])
    return R @ P


def _orbit(shape, n_proj, n_u, n_v, pitch, n_sub=1):
    ext = max(shape)
    return synth.circular_cone(n_proj, n_u, n_v, 3.0 * ext, 6.0 * ext, pitch, n_sub=n_sub)


# (volume, detector, projections, sub-views, pitch, roll, tilt): remainders of
# the 16 x 16 patch and of the column; volumes whose columns have 4, 8 and 16
# voxels; a truncated detector (footprints across every border, and patches
# that miss it); footprints too large for LDS (fine pitch); a rolled detector;
# a tilted one (a z coefficient in the depth row); fewer views than a round
CASES = [
    ((5, 17, 15), (30, 12), 3, 1, 1.4, 0.0, 0.0),
    ((70, 90, 100), (60, 33), 6, 1, 1.5, 0.0, 0.0),
    ((133, 130, 129), (96, 80), 5, 1, 1.5, 0.0, 0.0),
    ((37, 33, 20), (200, 230), 4, 2, 0.3, 0.0, 0.0),
    ((37, 33, 20), (40, 50), 7, 1, 1.5, 20.0, 0.0),
    ((129, 128, 128), (90, 70), 5, 1, 2.0, -7.0, 0.0),
    ((40, 41, 42), (50, 50), 4, 3, 1.5, 5.0, 9.0),
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("case", CASES)
def test_back_voxel_matches_oracle(case, dtype):
    shape, (n_u, n_v), n_proj, n_sub, pitch, roll, tilt = case
    P = _orbit(shape, n_proj, n_u, n_v, pitch, n_sub)
    if roll:
        P = _roll(P, roll)
    if tilt:
        a = np.radians(tilt)
        T = np.eye(4)
        T[1:3, 1:3] = [[np.cos(a), -np.sin(a)], [np.sin(a), np.cos(a)]]
        P = P @ T
    rng = np.random.default_rng(n_u)
    s = torch.from_numpy(rng.normal(0.5, 1.0, (n_proj, n_v, n_u)).astype(np.float32)).to(dtype)
    g = Geometry(P, n_u, n_v, shape)
    z = g.back_voxel(s.cuda())
    assert _rel(z.cpu().numpy(), oracle.back_voxel(P, shape, n_u, n_v, s.double().numpy())) <= TOL
    v = [n_proj - 1, 0, n_proj - 1]
    z2 = torch.ones_like(z)
    g.back_voxel(s[v].contiguous().cuda(), views=v, out=z2, accumulate=True)
    ref = 1.0 + oracle.back_voxel(P, shape, n_u, n_v, s[v].double().numpy(), views=v)
    assert _rel(z2.cpu().numpy(), ref) <= TOL


@pytest.mark.parametrize("grid", [(9, 40, 5), (20, 7, 33), (33, 150, 24), (40, 3, 18)])
def test_back_cylinder_matches_oracle(grid):
    """Patches of 16 angles spanning from a few degrees to the whole turn."""
    n_z, n_phi, n_r = grid
    ext = max(2 * n_r, n_z)
    P = synth.circular_cone(6, 44, 40, 3.0 * ext, 6.0 * ext, 2.4 * ext / 44)
    s = np.random.default_rng(n_r).normal(0.5, 1.0, (6, 40, 44)).astype(np.float32)
    g = CylinderGeometry(P, 44, 40, n_r, n_phi, n_z)
    z = g.back(torch.from_numpy(s).cuda()).cpu().numpy()
    ref = oracle.back_voxel_cyl(P, (n_r, n_phi, n_z, 1.0, 1.0), 44, 40, s.astype(np.float64))
    assert _rel(z, ref) <= TOL
