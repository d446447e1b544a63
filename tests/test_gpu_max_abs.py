"""The largest |r| of a backprojection wherever it lies: in each of the four
elements of a thread's pass, in the remainder and at the end.  One pixel is
nonzero, and every ray meets the volume, so missing it would leave the result
zero or scaled wrongly.
"""

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_30166_amd import Geometry

pytestmark = pytest.mark.gpu

# below one workgroup of 256 x 4, an odd size, and past 2048 of them
CASES = [((5, 7, 9), (11, 3), 2), ((33, 31, 35), (37, 41), 5), ((129, 130, 128), (421, 337), 15)]


@pytest.mark.parametrize("shape,det,n_proj", CASES)
def test_one_pixel_at_every_place(shape, det, n_proj):
    (n_u, n_v), ext = det, max(shape)
    # a detector half as wide as the volume's image
    P = synth.circular_cone(n_proj, n_u, n_v, 3.0 * ext, 6.0 * ext, ext / n_u)
    g = Geometry(P, n_u, n_v, shape, 1.0)
    n = n_proj * n_v * n_u
    stride = 256 * min((n + 1023) // 1024, 2048)   # threads of the launch
    at = {0, 1, 255, stride - 1, stride, 2 * stride + 3, 3 * stride, 4 * stride - 1, 4 * stride, n - 2,
          n - 1}
    for i in sorted(a for a in at if a < n):
        s = torch.zeros(n, device="cuda")
        s[i] = 2.0 ** 40
        big = g.back(s.view(n_proj, n_v, n_u))
        s[i] = 1.0
        one = g.back(s.view(n_proj, n_v, n_u))
        assert torch.equal(big, one * 2.0 ** 40)
        view, pix = divmod(i, n_v * n_u)
        ray = np.zeros((1, n_v, n_u))
        ray[0].flat[pix] = 1.0
        ref = oracle.back(P, shape, n_u, n_v, ray, 1.0, views=[view])
        assert ref.any()
        assert np.linalg.norm(one.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
