"""Demodulation on the FP32 matrix cores: the same chains of FMAs as on the
vector units, so the two agree bit for bit, and both match the oracle.

Which unit runs a call follows from the filter and the number of outputs, so a
frame with many traces takes the matrix cores where its first traces alone
take the vector units.
"""
import numpy as np
import pytest

import oracle
import paper_2512_11086_amd as bfm

pytestmark = pytest.mark.gpu


def _taps(n, cplx, seed):
    rng = np.random.default_rng(seed)
    h = rng.normal(size=n) / n
    return h + 1j * rng.normal(size=n) / n if cplx else h


@pytest.mark.parametrize("S, D, n_taps, cplx, r, out", [
    (1024, 1, 36, False, 0.25, "i16"),     # real and imaginary taps (quarter turns)
    (2051, 2, 36, True, 0.25, "f32"),      # odd rows: 2-byte aligned loads
    (2048, 2, 17, False, 0.25, "f32"),
    (2049, 2, 60, False, 0.2, "i16"),
])
def test_matrix_cores_equal_vector_units(dev, S, D, n_taps, cplx, r, out):
    import torch
    n_out = (S + D - 1) // D
    n = -(-(1 << 23) // n_out) + 1
    x = torch.randint(-32768, 32768, (n, S), dtype=torch.int16, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(S))
    h = _taps(n_taps, cplx, S)
    many = bfm.Demod(n, S, h, r * 30e6, 30e6, decimation=D, out=out)(x)
    few = bfm.Demod(100, S, h, r * 30e6, 30e6, decimation=D, out=out)(x[-100:].clone())
    assert torch.equal(many[-100:], few)


@pytest.mark.parametrize("n_tr, S, D, n_taps, cplx", [
    (1, 1, 1, 61, True), (15, 63, 1, 64, False), (16, 64, 1, 80, True), (17, 65, 1, 166, False),
    (3, 127, 2, 166, True), (33, 258, 2, 61, False), (5, 700, 3, 4, False), (2, 1000, 3, 166, True),
    (18, 517, 4, 1, False), (4, 900, 5, 255, True), (16, 260, 8, 1024, False),
    (3, 4100, 16, 3, False), (2, 300, 16, 500, True), (700, 2500, 1, 100, False),
])
def test_matrix_core_sizes_match_oracle(dev, n_tr, S, D, n_taps, cplx):
    import torch
    x = np.random.default_rng(S).integers(-30000, 30000, (n_tr, S)).astype(np.int16)
    h = _taps(n_taps, cplx, n_taps)
    got = bfm.Demod(n_tr, S, h, 6.1e6, 30e6, decimation=D, out="f32")(torch.from_numpy(x).cuda())
    rows = np.arange(n_tr) if n_tr < 50 else np.array([0, 1, n_tr // 2, n_tr - 1])
    ref = oracle.demod(x[rows], h, 6.1e6, 30e6, D)
    g = got.cpu().numpy()[rows].astype(np.float64)
    # FP32 sums of n_taps products: (n_taps + 4) roundings of at most the
    # largest sum of magnitudes
    bound = (n_taps + 4) * 6e-8 * 30000 * np.abs(h).sum()
    assert np.abs(g[..., 0] + 1j * g[..., 1] - ref).max() <= bound
