"""Warped projector pair: displacement nodes held per lane (forward) and per
brick in LDS (back), or read from memory where a brick's nodes do not fit,
against the FP64 oracle (relative L2 <= 1e-5, as for the unwarped pair: a
displacement errs by FP32 rounding, about 1e-6 voxel).
"""

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_30166_amd import Geometry

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b)


# (volume, grid (gz, gy, gx), displacement in voxels, sub-views, step): the
# coarsest grid; cells of several voxels; cells smaller than a voxel (a brick's
# nodes exceed the LDS); a grid finer along one axis only; bricks with a
# remainder of one voxel; displacements larger than a brick's halo; long steps
CASES = [
    ((17, 33, 40), (2, 2, 2), 2.0, 1, 0.5),
    ((20, 33, 65), (5, 4, 9), 3.0, 2, 0.5),
    ((18, 20, 34), (30, 25, 40), 1.5, 1, 0.5),
    ((16, 34, 33), (3, 60, 3), 2.5, 1, 0.5),
    ((33, 17, 33), (6, 6, 6), 7.0, 3, 0.8),
    ((24, 24, 24), (4, 5, 6), 2.0, 1, 3.0),
]


@pytest.mark.parametrize("case", CASES)
def test_warped_pair_matches_oracle(case):
    shape, grid, amp, n_sub, step = case
    n_u, n_v, n_proj = 41, 37, 6
    ext = max(shape)
    P = synth.circular_cone(n_proj, n_u, n_v, 3.0 * ext, 6.0 * ext, 2.6 * ext / n_u, n_sub=n_sub)
    rng = np.random.default_rng(grid[1])
    # smooth along the grid, so that neighbouring samples stay ordered
    z, y, x = np.meshgrid(*[np.linspace(0.0, 1.0, g) for g in grid], indexing="ij")
    U = np.stack([amp * np.cos(2.0 * (k + 1) * x + 3.0 * y - 2.0 * z + k) for k in range(3)], -1)
    U = U.astype(np.float32)
    tau = rng.uniform(-1.0, 1.0, (n_proj, n_sub))
    tau[0, 0] = 0.0
    g = Geometry(P, n_u, n_v, shape, step, U=U, tau=tau)
    v = rng.uniform(0.0, 1.0, shape).astype(np.float32)
    s = rng.normal(0.0, 1.0, (n_proj, n_v, n_u)).astype(np.float32)
    y_ref = oracle.forward(P, shape, n_u, n_v, v.astype(np.float64), step, U=U, tau=tau)
    z_ref = oracle.back(P, shape, n_u, n_v, s.astype(np.float64), step, U=U, tau=tau)
    y = g.forward(torch.from_numpy(v).cuda())
    zt = g.back(torch.from_numpy(s).cuda())
    assert _rel(y.cpu().numpy(), y_ref) <= 1e-5
    assert _rel(zt.cpu().numpy(), z_ref) <= 1e-5
    assert torch.equal(zt, g.back(torch.from_numpy(s).cuda()))   # bitwise reproducible
