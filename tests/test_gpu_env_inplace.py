"""An envelope written over its own image equals the one written beside it.

Each launch form reads a column before it stores any of it, so the two agree
bit for bit; the circulant product with few columns (an image of less than 256
groups of 16) is the form that spreads a column over workgroups when the
buffers are apart.
"""
import pytest

import paper_2512_11086_amd as bfm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (3, 96), (16, 192), (5, 251), (33, 999), (1, 1000),        # circulant, spread over workgroups
    (4100, 96),                                                # circulant, whole columns
    (9, 64), (130, 256), (4, 512), (2, 2048), (3, 7),          # the other forms
    (65, 130, 256),                                            # maximum in a pass of its own
])
@pytest.mark.parametrize("compress", ["none", "log"])
def test_envelope_over_its_image(dev, shape, compress):
    import torch
    x = torch.randn(shape, generator=torch.Generator().manual_seed(7)).cuda()
    env = bfm.Envelope(shape)
    want = env(x, compress=compress)
    for _ in range(3):
        y = x.clone()
        assert torch.equal(env(y, compress=compress, out=y), want)
