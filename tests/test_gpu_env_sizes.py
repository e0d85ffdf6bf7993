"""Envelope over the launch forms of its transforms: the tile FFT (64 to 256),
the FFT across lanes (512, 1024), the circulant product (other sizes, columns
spread over workgroups or not), the direct sum, and the compression by the
image's own maximum in each.

Tolerance: 1e-5 of the image's maximum, as for the envelope elsewhere; 1e-3 dB
(5e-5 relative where the envelope is above -60 dB, where an error of 1e-6 of
a value is 1e-5 dB) on the log scale within 60 dB.
"""
import numpy as np
import pytest
from scipy.signal import hilbert

import paper_2512_11086_amd as bfm

pytestmark = pytest.mark.gpu


def _image(shape, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal(shape) * np.exp(rng.standard_normal(shape[:-1] + (1,)))
    return x.astype(np.float32)


def _check(torch, shape, seed=0):
    x = _image(shape, seed)
    ref = np.abs(hilbert(x.astype(np.float64), axis=-1))
    t = torch.from_numpy(x).cuda()
    env = bfm.Envelope(shape)
    got = env(t).cpu().numpy()
    m = ref.max()
    assert np.abs(got - ref).max() <= 1e-5 * m
    log = env(t, compress="log", param=60.0).cpu().numpy()
    want = np.maximum(20 * np.log10(np.maximum(ref, 1e-30) / m), -60.0)
    near = ref > 1e-2 * m
    assert np.abs(log - want)[near].max() <= 1e-3
    assert log.min() >= -60.0 and log.max() <= 1e-3
    power = env(t, compress="power", param=0.5, ref=float(m) / 2).cpu().numpy()
    assert np.abs(power - np.minimum(2 * ref / m, 1.0) ** 0.5)[near].max() <= 1e-4
    fixed = env(t, compress="log", param=60.0, ref=float(m)).cpu().numpy()
    assert np.abs(fixed - want)[near].max() <= 1e-3


@pytest.mark.parametrize("shape", [
    (1, 64), (7, 64), (17, 64), (33, 128), (15, 256), (8, 256), (3, 512), (9, 1024),     # FFTs
    (1, 2048), (5, 32), (3, 7), (2, 23),                    # LDS FFT, direct sum
    (1, 24), (3, 25), (17, 31), (16, 96), (33, 100), (5, 101), (1, 192), (40, 251), (3, 999), (2, 1000),
    (2, 1001), (70, 60, 250), (65, 64, 33),                 # circulant, split and whole columns
    (97, 96, 64), (41, 101, 256), (91, 91, 256),            # workgroups of one and four wavefronts
])
def test_envelope_sizes(dev, shape):
    import torch
    _check(torch, shape, seed=sum(shape))


@pytest.mark.parametrize("shape", [(129, 128, 128), (128, 65, 256)])
def test_envelope_two_passes_over_the_image(dev, shape):
    import torch
    _check(torch, shape)


@pytest.mark.parametrize("shape", [(40, 256), (128, 128, 128), (40, 100), (4097, 128)])
def test_zero_image_compresses_to_the_floor(dev, shape):
    import torch
    env = bfm.Envelope(shape)
    z = torch.zeros(shape, device="cuda")
    assert torch.all(env(z, compress="log", param=40.0) == -40.0)
    assert torch.all(env(z, compress="power", param=0.5) == 0.0)


def test_unaligned_output(dev):
    import torch
    x = torch.from_numpy(_image((9, 100), 1)).cuda()
    env = bfm.Envelope(x.shape)
    buf = torch.empty(901, device="cuda")
    got = env(x, compress="log", out=buf[1:].view(9, 100))
    assert torch.equal(got, env(x, compress="log"))
