"""The launch a plan gets on small grids (CPU, host code).

Workgroups go to the 8 XCDs by depth slab, so the XCD with most slabs sets how
many of them share a CU and how many rounds a launch takes (32 CUs per XCD, two
workgroups each beside the usual 80 KiB of LDS).
"""
import ctypes
import random

import numpy as np
import pytest

import paper_2512_11086_amd as bfm
from paper_2512_11086_amd import _lib

MM = 1e-3


def _launch(mode, cols, pitch, fs, n_tx, n_ch, dims, half, z, iq=False, e_type="f32", **kw):
    xdc = np.eye(4)
    xdc[0, 3] = xdc[1, 3] = (cols - 1) / 2 * pitch
    y = 0.0 if mode == "forces" else half
    d = dict(mode=mode, n_tx=n_tx, n_ch=n_ch, n_samples=1500, n_elem=(cols, cols),
             pitch=(pitch, pitch), xdc=xdc, fs=fs, fc=fs / 4, c=1540.0, t0=0.0, f_number=1.0,
             interp="cubic", dims=dims, gmin=(-half, -y, z[0]), gmax=(half, y, z[1]), iq=iq,
             tx_elements=(np.arange(n_tx) * cols // n_tx).astype(np.int32),
             channel_map=(np.arange(n_ch) * cols // n_ch).astype(np.int32))
    if mode == "tpw":
        d["tx_angles"] = np.deg2rad(np.linspace(-10, 10, n_tx))
    d.update(kw)
    out = _lib.TestLaunch()
    m = bfm.params_from_desc(d, None, e_type)
    _lib.check(_lib.lib().bf_test_das_launch(ctypes.byref(m.p), 3, ctypes.byref(out)))
    return out


def _per_xcd(o):
    return o.blocks[0] * o.blocks[1] * -(-o.blocks[2] // 8) * o.groups


def test_batches_fill_a_cu_only_where_each_has_one_workgroup():
    rng = random.Random(4)
    larger = crowded = 0
    for _ in range(1500):
        mode = rng.choice(["forces", "forces", "tpw", "vls"])
        cols, pitch, fs = rng.choice([(32, 0.2 * MM, 20e6), (64, 0.2 * MM, 30e6), (128, 0.1 * MM, 30e6)])
        dims = ((rng.randint(60, 400), 1, rng.randint(60, 300)) if mode == "forces" else
                (rng.randint(16, 64), rng.randint(16, 64), rng.randint(24, 128)))
        iq = mode == "forces" and rng.random() < 0.4
        o = _launch(mode, cols, pitch, fs / (2 if iq else 1), rng.choice([8, 12, 20, 24, 32]),
                    rng.randint(cols // 2, cols), dims, cols * pitch / 2 * rng.uniform(0.5, 1),
                    (4 * MM, 35 * MM), iq=iq, **(dict(focal_depth=-10 * MM) if mode == "vls" else {}))
        if not o.lds:
            continue
        windows = 2 * o.nb * o.lmax * 16 * (2 if iq else 1)
        if windows > 80 * 1024:
            assert _per_xcd(o) <= 32
            larger += 1
        crowded += o.blocks[0] * o.blocks[1] * o.blocks[2] * o.groups <= 256 < 8 * _per_xcd(o)
    assert larger > 50 and crowded > 50


def test_a_larger_batch_saves_one():
    """252 x 106 points: 36 workgroups on seven XCDs, two per CU (batches of 12, not 16)."""
    o = _launch("forces", 64, 0.2 * MM, 30e6, 24, 36, (252, 1, 106), 4.15 * MM, (5.6 * MM, 30 * MM),
                interp="linear")
    assert (list(o.blocks), o.groups, _per_xcd(o), o.nb) == ([4, 1, 7], 9, 36, 12)
    o = _launch("forces", 32, 0.2 * MM, 20e6, 32, 32, (128, 1, 128), 6.4 * MM, (5 * MM, 40 * MM))
    assert (_per_xcd(o), o.nb) == (16, 16)


# Splits that the whole launch's workgroups, rounded-down channel counts or a
# loop that began at two chunks had made too fine or too coarse: (description,
# smallest and largest number of groups that suits the XCDs' rounds).
CASES = [
    # 8 boxes per XCD: 8 groups are one round, 9 the start of another (152, 173 us)
    (("hercules", 128, 0.1 * MM, 30e6, 16, 116, (31, 31, 77), 6.4 * MM, (5 * MM, 30 * MM)), {}, 8, 8),
    # 16 groups 123 us, 11 (one workgroup more than a round) 132
    (("forces", 128, 0.1 * MM, 15e6, 12, 128, (113, 1, 272), 6.39 * MM, (4.6 * MM, 30 * MM)),
     dict(iq=True, interp="linear"), 16, 16),
    (("forces", 64, 0.2 * MM, 15e6, 24, 34, (257, 1, 335), 6.0 * MM, (5 * MM, 30 * MM)),
     dict(iq=True), 7, 9),
    # 11 chunks of 4 rows: one group per chunk is allowed
    (("forces", 64, 0.2 * MM, 15e6, 32, 42, (60, 1, 60), 6.0 * MM, (5 * MM, 14 * MM)),
     dict(iq=True), 11, 11),
    # half a workgroup per CU, or less, with one chunk a group
    (("tpw", 32, 0.2 * MM, 20e6, 16, 16, (24, 24, 48), 3.2 * MM, (4 * MM, 40 * MM)), {}, 4, 4),
    (("tpw", 32, 0.2 * MM, 20e6, 16, 8, (24, 24, 48), 3.2 * MM, (4 * MM, 40 * MM)), {}, 2, 2),
]


@pytest.mark.parametrize("args, kw, low, high", CASES)
def test_groups_follow_the_rounds_of_the_fullest_xcd(args, kw, low, high):
    o = _launch(*args, **kw)
    assert o.lds and low <= o.groups <= high


def test_float_volumes_do_not_split_further_than_their_aim():
    """Their images feed dL/dc; fewer groups only without mirror points."""
    box = dict(half=3.2 * MM, z=(4 * MM, 35 * MM))
    far = [_launch("hercules", 32, 0.2 * MM, 20e6, 16, 32, (65, 62, 85), e_type=t, **box).groups
           for t in ("f32", "i32")]
    assert far[0] == 2 < far[1]
    # 79 x 31 x 91 points, receivers off the centre: 3 groups 174 us, 4 198
    o = _launch("hercules", 128, 0.1 * MM, 30e6, 12, 76, (79, 31, 91), 5 * MM, (5 * MM, 30 * MM))
    assert (o.mirrors, o.groups) == (0, 3)
