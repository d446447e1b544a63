"""The streams beside the projectors (max |r|, the scaling of the integer
volume, the SIRT update): four elements per pass and a remainder, at sizes
below one workgroup, at odd ones and past the largest grid (2048 x 1024).
"""

import numpy as np
import pytest
import torch

import synth
from paper_2609_30166_amd import Geometry

pytestmark = pytest.mark.gpu

# (volume, detector (n_u, n_v), projections): the last has 2.15 M voxels and
# 2.13 M pixels, both past 2048 workgroups x 1024 elements
CASES = [((5, 7, 9), (11, 3), 2), ((33, 31, 35), (37, 41), 5), ((129, 130, 128), (421, 337), 15)]


def _geometry(shape, det, n_proj):
    ext = max(shape)
    P = synth.circular_cone(n_proj, det[0], det[1], 3.0 * ext, 6.0 * ext, 2.4 * ext / det[0])
    return Geometry(P, det[0], det[1], shape, 1.0)


@pytest.mark.parametrize("case", CASES)
def test_accumulate_adds_every_voxel(case):
    shape, det, n_proj = case
    g = _geometry(*case)
    gen = torch.Generator().manual_seed(3)
    r = torch.randn((n_proj, det[1], det[0]), generator=gen).cuda()
    old = torch.randn(shape, generator=gen).cuda()
    z = g.back(r)
    out = old.clone()
    g.back(r, out=out, accumulate=True)
    assert torch.equal(out, old + z)
    # the largest |r| wherever it lies (a thread's first to fourth element of a
    # pass, the remainder, the last element): sums scale with it exactly
    flat = r.view(-1)
    n = flat.numel()
    for at in (0, n // 4, n // 2, 3 * n // 4, n - 1):
        q = torch.zeros_like(flat)
        q[at] = 2.0 ** 40
        one = torch.zeros_like(flat)
        one[at] = 1.0
        a, b = g.back(q.view_as(r)), g.back(one.view_as(r))
        assert torch.isfinite(a).all() and torch.equal(a, b * 2.0 ** 40)


@pytest.mark.parametrize("nonneg", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_update_of_every_voxel(case, nonneg):
    shape, det, n_proj = case
    g = _geometry(*case)
    gen = torch.Generator().manual_seed(4)
    b = torch.randn((n_proj, det[1], det[0]), generator=gen).cuda()
    x0 = torch.randn(shape, generator=gen).cuda()
    x = x0.clone()
    g.sirt(x, b, 1, alpha=0.7, nonneg=nonneg)
    row = g.forward(torch.ones(shape, device="cuda"))
    col = g.back(torch.ones_like(b))
    r = torch.where(row > 0, (b - g.forward(x0)) / row, torch.zeros_like(b))
    c = torch.where(col > 0, 1.0 / col, torch.zeros_like(col))
    want = x0.double() + 0.7 * c.double() * g.back(r).double()
    if nonneg:
        want = want.clamp(min=0)
    # A ones is summed in another order than the row sums of the fused loop:
    # FP32 sums of some 100 samples, 1e-5 relative
    err = (x.double() - want).norm() / (want - x0.double()).norm()
    assert float(err) <= 1e-5, float(err)
