"""A view list of 2^19 entries on a one-tile detector: 2^19 workgroups of
work, far below the threads of a launch, however they are grouped.
"""

import numpy as np
import pytest
import torch

import synth
from paper_2609_30166_amd import Geometry

pytestmark = pytest.mark.gpu


def test_forward_over_a_long_list():
    n_proj, n = 64, 1 << 19
    P = synth.circular_cone(n_proj, 2, 2, 30.0, 60.0, 4.0)
    g = Geometry(P, 2, 2, (6, 6, 6))
    x = torch.from_numpy(np.random.default_rng(1).uniform(0, 1, g.shape).astype(np.float32)).cuda()
    views = np.random.default_rng(2).integers(0, n_proj, n).astype(np.int32)
    y = g.forward(x, views=views)
    assert g.sample_count(views) > 0
    one = g.forward(x)
    assert one.any()
    assert torch.equal(y, one[torch.from_numpy(views).long().cuda()])
