"""Forward projector: the pair-packed gather copies at the edges of their
32 x 32 tiles, rays entering through every face of the hull, and rays that
graze it.  Each case compares with the FP64 oracle on the same (rounded)
volume; FP32 sums of exactly placed samples are held to 1e-5 relative L2, as
everywhere else.
"""

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_30166_amd import Geometry

pytestmark = pytest.mark.gpu

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _orbit(shape, n_u, n_v, axis):
    """8 views around ``axis`` (0: x, 1: y, 2: z), so that rays enter through
    the faces across the other two."""
    ext = float(max(shape))
    src, views = 3.0 * ext, []
    for k in range(8):
        a = 2 * np.pi * (k + 0.3) / 8
        e = np.zeros(3)
        p, q = [i for i in range(3) if i != axis]
        e[p], e[q] = np.cos(a), np.sin(a)
        eu = np.zeros(3)
        eu[p], eu[q] = -np.sin(a), np.cos(a)
        ev = np.zeros(3)
        ev[axis] = 1.0
        views.append(synth.view_matrix(src * e, -src * e, eu, ev, 3.0 * ext / n_u, 3.0 * ext / n_v,
                                       n_u, n_v))
    return np.asarray(views)[:, None]


def _check(P, shape, n_u, n_v, dtype, views=None):
    rng = np.random.default_rng(5)
    x = torch.from_numpy(rng.uniform(0.0, 1.0, shape).astype(np.float32)).to(DTYPES[dtype])
    ref = oracle.forward(P, shape, n_u, n_v, x.double().numpy(), views=views)
    g = Geometry(P, n_u, n_v, shape)
    y = g.forward(x.cuda(), views=views).double().cpu().numpy()
    assert np.linalg.norm(y - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(2, 2, 2), (3, 31, 32), (2, 33, 65), (5, 64, 2), (33, 2, 34)])
def test_forward_at_tile_edges(shape, dtype):
    _check(_orbit(shape, 21, 19, 2), shape, 21, 19, dtype)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("views", [None, [5], [7, 0, 0, 3, 6, 2, 1, 4, 5]])
def test_forward_through_every_face(axis, views):
    _check(_orbit((20, 33, 27), 37, 35, axis), (20, 33, 27), 37, 35, "f32", views)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_forward_grazing_rays(dtype):
    """A source in the plane of a hull face: a row of rays runs inside the
    face (every sample's corner is clamped), its neighbours just inside and
    just outside."""
    # every entry of the matrices and their inverses is exact in binary, so
    # both sides place the centre row exactly in the face
    shape, n_u, n_v = (9, 17, 15), 25, 17
    views = []
    for s in (-1.0, 1.0):
        z = s * 0.5 * (shape[0] - 1)
        views.append(synth.view_matrix([64.0, 0, z], [-64.0, 0, z], [0, 1.0, 0], [0, 0, 1.0],
                                       2.0, 2.0 ** -10, n_u, n_v))
        y = s * 0.5 * (shape[1] - 1)
        views.append(synth.view_matrix([0, y, 64.0], [0, y, -64.0], [1.0, 0, 0], [0, 1.0, 0],
                                       2.0, 2.0 ** -10, n_u, n_v))
    P = np.asarray(views)[:, None]
    ones = oracle.forward(P, shape, n_u, n_v, np.ones(shape))
    assert (ones[:, n_v // 2, n_u // 2] > 0).all()   # the grazing rays count
    _check(P, shape, n_u, n_v, dtype)
