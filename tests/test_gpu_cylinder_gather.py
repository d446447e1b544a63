"""Cylindrical projector: the two pair-packed copies at the edges of their 32 x
32 tiles and across the angle's wrap, rays through and beside the axis, and
16-bit volumes (read without copies), against the FP64 oracle.  Relative L2 <=
1e-5: the FP32 polar map errs by about 1e-7 of the radius.
"""

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_30166_amd import CylinderGeometry

pytestmark = pytest.mark.gpu

GRIDS = [(3, 3, 2), (4, 31, 32), (5, 32, 33), (4, 33, 31), (6, 96, 40), (7, 200, 65)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("grid", GRIDS)
def test_forward_matches_oracle(grid, dtype):
    n_z, n_phi, n_r = grid
    ext = max(2 * n_r, n_z)
    P = synth.circular_cone(7, 41, 23, 3.0 * ext, 6.0 * ext, 4.2 * ext / 41, theta0=0.1)
    x = np.random.default_rng(n_phi).uniform(0.0, 1.0, grid).astype(np.float32)
    xt = torch.from_numpy(x).to(dtype)
    cyl = (n_r, n_phi, n_z, 1.0, 1.0)
    ref = oracle.forward_cyl(P, cyl, 41, 23, xt.double().numpy())
    g = CylinderGeometry(P, 41, 23, n_r, n_phi, n_z)
    y = g.forward(xt.cuda()).double().cpu().numpy()
    # the middle column's rays pass through the axis, where the angle has no
    # value: a sample there takes any of ring 0's (the oracle's own moves when
    # the geometry is shifted by 1e-13), so only its range is checked
    mid = np.arange(41) == 20
    assert np.linalg.norm((y - ref)[..., ~mid]) <= 1e-5 * np.linalg.norm(ref[..., ~mid])
    assert (y >= -1e-6).all() and (y <= 1.00001 * 2.0 * ext).all()


def test_sirt_matches_oracle():
    grid, cyl = (6, 70, 33), (33, 70, 6, 1.0, 1.0)
    P = synth.circular_cone(9, 40, 16, 200.0, 400.0, 4.0)
    x = np.random.default_rng(0).uniform(0.5, 1.0, grid)
    b = oracle.forward_cyl(P, cyl, 40, 16, x).astype(np.float32)
    g = CylinderGeometry(P, 40, 16, 33, 70, 6)
    v = torch.zeros(grid, device="cuda")
    g.sirt(v, torch.from_numpy(b).cuda(), 3)
    ref, _ = oracle.sirt_cyl(P, cyl, 40, 16, b.astype(np.float64), 3)
    assert np.linalg.norm(v.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
