"""Exact-transpose backprojector: work handed out in pixel blocks, owned
sample ranges and merged sums, at the sizes where they can go wrong, against
the FP64 oracle (relative L2 <= 1e-5: exact integer sums of FP32 weights).
"""

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_30166_amd import Geometry

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


# (volume, detector, projections, sub-views, step): bricks of 32 x 16 x 16 with
# remainders of one voxel and none, more and fewer (projection, sub-view) pairs
# than a batch of 64, fewer pixel blocks than waves, and a step so small that a
# lane's run of samples passes the merge limit of 1024
CASES = [
    ((16, 16, 32), (30, 21), 5, 1, 0.5),
    ((17, 33, 65), (50, 40), 7, 1, 0.5),
    ((18, 34, 66), (50, 40), 3, 3, 0.7),
    ((16, 17, 33), (5, 3), 2, 1, 0.5),
    ((20, 12, 9), (16, 16), 130, 1, 0.5),
    ((11, 19, 40), (24, 24), 33, 2, 0.5),
    ((16, 16, 32), (12, 12), 3, 1, 0.01),
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("case", CASES)
def test_back_matches_oracle(case, dtype):
    shape, (n_u, n_v), n_proj, n_sub, step = case
    ext = max(shape)
    P = synth.circular_cone(n_proj, n_u, n_v, 3.0 * ext, 6.0 * ext, 2.4 * ext / n_u, n_sub=n_sub)
    rng = np.random.default_rng(n_proj)
    s = rng.normal(0.0, 1.0, (n_proj, n_v, n_u)).astype(np.float32)
    s[:, n_v // 2] *= 20.0   # rays that may not merge next to rays that may
    s[0, :, : n_u // 3] = 0.0
    st = torch.from_numpy(s).to(dtype)
    ref = oracle.back(P, shape, n_u, n_v, st.double().numpy(), step)
    g = Geometry(P, n_u, n_v, shape, step)
    z = g.back(st.cuda())
    assert _rel(z.double().cpu().numpy(), ref) <= 1e-5
    assert torch.equal(z, g.back(st.cuda()))   # bitwise reproducible
    v = list(range(0, n_proj, 2)) + [0]
    zv = g.back(st[v].contiguous().cuda(), views=v).double().cpu().numpy()
    assert _rel(zv, oracle.back(P, shape, n_u, n_v, st[v].double().numpy(), step, views=v)) <= 1e-5


def test_back_of_constant_and_non_finite_images():
    shape, n_u, n_v = (16, 16, 40), 20, 18
    P = synth.circular_cone(6, n_u, n_v, 120.0, 240.0, 4.0)
    g = Geometry(P, n_u, n_v, shape)
    ones = torch.ones(6, n_v, n_u, device="cuda")
    ref = oracle.back(P, shape, n_u, n_v, np.ones((6, n_v, n_u)))
    assert _rel(g.back(ones).double().cpu().numpy(), ref) <= 1e-5
    assert not g.back(torch.zeros_like(ones)).any()
    for bad in (float("nan"), float("inf")):
        s = ones.clone()
        s[2, 3, 4] = bad
        assert torch.isnan(g.back(s)).all()
    # the lowest and largest finite values neither overflow nor vanish
    for c in (1e-30, 1e30):
        z = g.back(ones * c).double().cpu().numpy()
        assert _rel(z, ref * np.float64(np.float32(c))) <= 1e-5
