"""The 32 -> 16 convolution on volumes of 384 tiles of four planes, above and
below, where the tile has four planes or two, of one tensor and of a
concatenation, against FP64 (FP32 outputs of BF16 inputs: 1e-5 relative, as for
the other shapes).
"""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _vp(t):
    return ctypes.c_void_p(t.data_ptr())


@pytest.mark.parametrize("cat", [False, True])
@pytest.mark.parametrize("shape", [(48, 56, 64), (48, 64, 64), (45, 50, 96), (62, 61, 64)])
def test_conv3_32_to_16(shape, cat):
    from paper_2609_30166_amd import _lib

    L = _lib.lib()
    c = ctypes.c_void_p()
    assert L.ctrex_create(ctypes.byref(c), 0) == 0
    gen = torch.Generator().manual_seed(7)
    x = torch.randn(shape + (32,), generator=gen).bfloat16()
    w = (0.1 * torch.randn(16, 32, 27, generator=gen)).bfloat16().float()
    b = torch.randn(16, generator=gen)
    wd, bd = w.cuda(), b.cuda()
    wt = torch.empty(27 * 32 * 16, dtype=torch.bfloat16, device="cuda")
    wb = torch.empty_like(wt)
    assert L.ctrex_nn_pack_conv3(c, _vp(wd), 16, 32, _vp(wt), _vp(wb), None) == 0
    out = torch.empty(shape + (16,), device="cuda")
    if cat:
        lo, hi = x[..., :16].contiguous().cuda(), x[..., 16:].contiguous().cuda()
        code = L.ctrex_nn_conv3_cat(c, _vp(lo), 16, 0, 16, _vp(hi), 16, 0, 16, _vp(wt), _vp(bd),
                                    _vp(out), 16, 0, 16, None, 0, 0, 0, None, 0, 0, *shape,
                                    _lib.NN_OUT_F32, None)
    else:
        xd = x.cuda()
        code = L.ctrex_nn_conv3(c, _vp(xd), 32, 0, 32, _vp(wt), _vp(bd), _vp(out), 16, 0, 16, *shape,
                                _lib.NN_OUT_F32, None)
    assert code == 0
    ref = torch.nn.functional.conv3d(x.double().permute(3, 0, 1, 2)[None],
                                     w.double().view(16, 32, 3, 3, 3), b.double(), padding=1)
    ref = ref[0].permute(1, 2, 3, 0).numpy()
    got = out.double().cpu().numpy()
    L.ctrex_destroy(c)
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
