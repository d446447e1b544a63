"""Backprojector with steps so small that the 64 rays of a pixel block have
more than 2^25 samples in a brick, so a lane's share of them times 64 does not
fit 32 bits.  Against the FP64 oracle, relative L2 <= 1e-5 (at most 1024 FP32
additions before an exact integer sum).
"""

import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_30166_amd import Geometry

pytestmark = pytest.mark.gpu

SHAPE, N, STEP = (16, 16, 32), 8, 5e-5


def _direct(g, s):
    from paper_2609_30166_amd._lib import check, lib

    out = torch.empty(g.shape, dtype=torch.float32, device=g.device)
    check(g._ctx, lib().ctrex_back_project_noalloc(
        g._ctx, ctypes.c_void_p(s.data_ptr()), 0, ctypes.c_void_p(out.data_ptr()), 0, None, 0,
        ctypes.c_void_p(torch.cuda.current_stream(g.device).cuda_stream)))
    return out


@pytest.mark.parametrize("form", ["owner", "direct", "warp", "warp, fine grid"])
def test_back_with_a_tiny_step(form):
    # 64 rays along x through the one brick, each with about 31 / STEP samples
    assert 63 * 64 * 30 / STEP > 2 ** 31
    P = synth.view_matrix([96.0, 1.3, 0.7], [-96.0, 0.4, -0.2], [0, 1.0, 0], [0, 0, 1.0], 2.0, 2.0,
                          N, N)[None, None]
    s = np.random.default_rng(1).uniform(0.5, 1.0, (1, N, N)).astype(np.float32)
    U = tau = None
    if form.startswith("warp"):
        # 15 nodes per axis are more than a workgroup keeps in LDS
        k = 15 if form.endswith("grid") else 3
        U = synth.smooth_displacement(k, 1.5, np.random.default_rng(2))
        tau = np.ones((1, 1))
    g = Geometry(P, N, N, SHAPE, STEP, U=U, tau=tau)
    st = torch.from_numpy(s).cuda()
    z = (_direct(g, st) if form == "direct" else g.back(st)).double().cpu().numpy()
    ref = oracle.back(P, SHAPE, N, N, s.astype(np.float64), STEP, U=U, tau=tau)
    assert np.linalg.norm(z - ref) <= 1e-5 * np.linalg.norm(ref)
