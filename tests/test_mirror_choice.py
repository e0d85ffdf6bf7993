"""Mirror points never cost a HERCULES plan its LDS kernel (CPU, host code).

The launch is chosen among the plain one and those over the geometry's mirror
axes; a launch whose windows, guard or tables leave no room for the mirror
copies has to fall back to fewer copies, and to the gather kernel only where
the plain launch does not fit either.
"""
import ctypes
import math
import random

import numpy as np
import pytest

import paper_2512_11086_amd as bfm
from paper_2512_11086_amd import _lib


def _launch(desc, allowed):
    out = _lib.TestLaunch()
    m = bfm.params_from_desc(desc, None)
    _lib.check(_lib.lib().bf_test_das_launch(ctypes.byref(m.p), allowed, ctypes.byref(out)))
    return out


def _desc(n_tx, n_ch, pitch, fs, dims, half, z, iq=False, **kw):
    xdc = np.eye(4)
    xdc[0, 3], xdc[1, 3] = (n_tx - 1) / 2 * pitch, (n_ch - 1) / 2 * pitch
    d = dict(mode="hercules", n_tx=n_tx, n_ch=n_ch, n_samples=1024, n_elem=(n_tx, n_ch),
             pitch=(pitch, pitch), xdc=xdc, fs=fs, fc=fs / 4, c=1540.0, t0=0.0, f_number=1.0,
             interp="cubic", dims=dims, gmin=(-half[0], -half[1], z[0]),
             gmax=(half[0], half[1], z[1]), iq=iq)
    d.update(kw)
    return d


def test_symmetric_plans_keep_the_lds_kernel():
    rng = random.Random(11)
    used = {0: 0, 1: 0, 2: 0, 3: 0}
    for _ in range(1500):
        n_tx = rng.choice([32, 64, 128, 256])
        n_ch = rng.choice([n_tx, n_tx, 256, 512, 1024])
        pitch, fs = rng.choice([0.1, 0.2, 0.3, 0.4]) * 1e-3, rng.choice([10e6, 20e6, 30e6, 40e6])
        dims = (rng.randint(8, 160), rng.randint(8, 160), rng.randint(2, 256))
        half = (rng.uniform(0.3, 1) * n_tx * pitch / 2, rng.uniform(0.3, 1) * n_ch * pitch / 2)
        z0 = rng.uniform(2e-3, 8e-3)
        kw = dict(focal_depth=-rng.uniform(5e-3, 30e-3)) if rng.random() < 0.3 else {}
        d = _desc(n_tx, n_ch, pitch, fs, dims, half, (z0, z0 + rng.uniform(5e-3, 60e-3)),
                  iq=rng.random() < 0.3, f_number=rng.choice([0.0, 0.5, 1.0, 1.5]),
                  interp=rng.choice(["cubic", "linear"]), **kw)
        plain, chosen = _launch(d, 0), _launch(d, 3)
        assert chosen.lds or not plain.lds, d
        used[chosen.mirrors] += 1
    assert min(used.values()) > 50      # (the geometries do exercise every choice)


@pytest.mark.parametrize("desc", [
    # windows longer than a copy's set
    _desc(128, 128, 0.2e-3, 20e6, (64, 64, 128), (12.8e-3, 12.8e-3), (5e-3, 50e-3), iq=True),
    # tables of a large aperture
    _desc(128, 768, 0.1e-3, 30e6, (128, 128, 256), (6.4e-3, 38.4e-3), (5e-3, 30e-3)),
    _desc(256, 512, 0.1e-3, 30e6, (128, 128, 256), (6.4e-3, 6.4e-3), (5e-3, 30e-3)),
    # guard of a coarse lateral grid without apodization limits
    _desc(256, 256, 0.1e-3, 30e6, (64, 64, 256), (12.8e-3, 12.8e-3), (5e-3, 30e-3)),
])
def test_launches_that_do_not_fit_mirrored(desc):
    plain, chosen = _launch(desc, 0), _launch(desc, 3)
    assert plain.lds and plain.mirrors == 0
    assert chosen.lds and chosen.nb >= 1


def test_headline_volume_mirrors_both_axes():
    d = _desc(128, 128, 0.1e-3, 30e6, (128, 128, 256), (6.4e-3, 6.4e-3), (5e-3, 30e-3))
    got = _launch(d, 3)
    assert got.lds and got.mirrors == 3 and (got.nb, got.zp) == (15, 1)
    assert math.prod(got.block) == 12 and tuple(got.tile) == (8, 8, 1)


def test_real_data_boxes_keep_the_bits_of_a_position():
    """FP32 positions relative to the middle of a box's delays lose bits as these
    spread: a box deeper than the default's 6 depths stays within 16 samples of its
    reference, or has one for every 4 depths at most."""
    rng = random.Random(3)
    shapes, rows = set(), 0
    for _ in range(600):
        n = rng.choice([32, 64, 128])
        half = rng.uniform(0.3, 1) * n * 0.1e-3
        d = _desc(n, n, 0.2e-3, rng.choice([20e6, 30e6]),
                  (rng.randint(16, 128), rng.randint(16, 128), rng.randint(4, 256)), (half, half),
                  (5e-3, rng.uniform(15e-3, 45e-3)))
        if rng.random() < 0.5:
            d["channel_map"] = np.roll(np.arange(n), 1)       # no mirror in y
        got = _launch(d, rng.choice([0, 3]))
        depths = got.tile[2] * got.block[2] * got.zp
        step = 2 * d["fs"] / d["c"] * (d["gmax"][2] - d["gmin"][2]) / (d["dims"][2] - 1)
        near = depths <= 6 or step * (depths - 1) / 2 <= 16
        assert got.refs == (1 if near else got.block[2]), d
        assert near or got.tile[2] * got.zp <= 4, d
        rows += got.refs > 1
        shapes.add((tuple(got.tile), tuple(got.block)))
    assert len(shapes) > 2 and rows
