"""Sharpness loss and gradient over its launch forms: one workgroup per image
(with and without 16-byte loads), and images split over workgroups.

Sums are FP64 and the outputs are rounded once to FP32 (6e-8); 1e-6 leaves
room for the FP64 evaluation of the gradient's two terms.
"""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2512_11086_amd as bfm
from paper_2512_11086_amd import _lib
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu
TOL = 1e-6


def _check(x, loss, g):
    for f in range(x.shape[0]):
        L, gr = oracle.sharpness(x[f].astype(np.float64), grad=True)
        assert abs(float(loss[f]) - L) <= TOL * max(abs(L), 1e-30)
        if g is not None:
            assert rel_l2(g[f].cpu().numpy(), gr) <= TOL


@pytest.mark.parametrize("images, n", [(1, 1), (3, 63), (2, 8191), (3, 32769), (2, 65536),
                                       (2, 131071), (1, 131072), (3, 131073), (2, 221185),
                                       (1, 1 << 20)])
def test_sharpness_sizes(dev, images, n):
    import torch
    x = np.random.default_rng(n).standard_normal((images, n)).astype(np.float32)
    t = torch.from_numpy(x).cuda()
    _check(x, *bfm.sharpness(t))
    _check(x, bfm.sharpness(t, grad=False), None)


def test_sharpness_zero_image_split(dev):
    import torch
    x = np.zeros((2, 140000), dtype=np.float32)
    x[1, 7] = 2.0
    loss, g = bfm.sharpness(torch.from_numpy(x).cuda())
    assert float(loss[0]) == 0.0 and float(loss[1]) == -1.0
    assert not g.any()


def test_sharpness_gradient_over_the_image(dev):
    import torch
    x = np.random.default_rng(4).standard_normal((2, 150001)).astype(np.float32)
    t = torch.from_numpy(x).cuda()
    loss = torch.empty(2, device="cuda")
    p = ctypes.c_void_p
    s = p(torch.cuda.current_stream().cuda_stream)
    _lib.check(_lib.lib().bf_sharpness(p(t.data_ptr()), x.shape[1], 2, p(loss.data_ptr()),
                                       p(t.data_ptr()), s))
    _check(x, loss, t)
