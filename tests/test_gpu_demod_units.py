"""Demodulation on the vector units and on the matrix cores: the same chains of
FMAs, so the two agree bit for bit wherever both can run; and which of them a
call takes.

The unit is set per demodulator and reported back, so each side is known to have
run on the unit it names.
"""
import numpy as np
import pytest

import paper_2512_11086_amd as bfm
from paper_2512_11086_amd import _lib

pytestmark = pytest.mark.gpu
VECTOR, MATRIX = 1, 2


def _taps(n, cplx):
    rng = np.random.default_rng(n)
    h = rng.normal(size=n) / n
    return h + 1j * rng.normal(size=n) / n if cplx else h


@pytest.mark.parametrize("n_tr, S, D, n_taps, cplx, r, out", [
    (33, 2051, 1, 61, True, 0.25, "f32"), (17, 2816, 2, 166, True, 0.25, "i16"),
    (16, 2816, 1, 166, False, 0.2, "i16"), (5, 901, 2, 61, False, 0.2, "f32"),
    (1, 1, 1, 1, True, 0.25, "f32"), (40, 333, 3, 4, False, 0.25, "i16"),
    (18, 517, 4, 1, True, 0.2, "f32"), (3, 700, 5, 255, True, 0.25, "f32"),
    (15, 1000, 12, 49, False, 0.2, "i16"), (16, 260, 16, 24, True, 0.25, "f32"),
    (2000, 300, 6, 6, False, 0.25, "f32"), (9, 4096, 8, 1024, True, 0.2, "f32"),
])
def test_matrix_cores_equal_vector_units(dev, n_tr, S, D, n_taps, cplx, r, out):
    import torch
    x = torch.randint(-32768, 32768, (n_tr, S), dtype=torch.int16, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(S))
    d = bfm.Demod(n_tr, S, _taps(n_taps, cplx), r * 30e6, 30e6, decimation=D, out=out)
    got = {}
    for unit in (VECTOR, MATRIX):
        assert _lib.lib().bf_test_demod_unit(d._h, unit) == unit
        got[unit] = d(x)
    assert torch.equal(got[VECTOR], got[MATRIX])


@pytest.mark.parametrize("n_tr, S, D, n_taps, unit", [
    (16384, 2816, 2, 166, MATRIX), (16384, 2816, 4, 36, MATRIX), (4800, 300, 6, 6, MATRIX),
    (4096, 2048, 2, 36, VECTOR),
    # few traces, or long records with few taps, at D >= 3: bound by a workgroup's latency
    (194, 1501, 12, 49, VECTOR), (78, 1000, 16, 31, VECTOR), (814, 2048, 16, 13, VECTOR),
    (1588, 2816, 3, 22, VECTOR), (1026, 2816, 4, 1, VECTOR),
])
def test_unit_by_size(dev, n_tr, S, D, n_taps, unit):
    d = bfm.Demod(n_tr, S, _taps(n_taps, False), 7.5e6, 30e6, decimation=D)
    assert _lib.lib().bf_test_demod_unit(d._h, 0) == unit
