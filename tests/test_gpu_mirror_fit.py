"""Symmetric HERCULES plans whose mirror copies do not (all) fit LDS: the LDS
kernel runs with fewer copies or none, and the image is the oracle's to the
1e-5 relative L2 of the DAS tests."""
import numpy as np
import pytest

import oracle
import paper_2512_11086_amd as bfm
from paper_2512_11086_amd import _lib
from synth.configs import MM, describe
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu


def _desc(n_tx, n_ch, pitch, fs, S, dims, half, z, **kw):
    return describe("hercules", (n_tx, n_ch), (pitch, pitch), n_tx, n_ch, S, fs, fs / 4, dims,
                    (-half[0], -half[1], z[0]), (half[0], half[1], z[1]), t0=0.0,
                    **dict(dict(f_number=1.0, interp="cubic"), **kw))


@pytest.mark.parametrize("desc, iq, most", [
    # windows of 400 quads and more: longer than a copy's set in x and y
    (_desc(24, 24, 1.6 * MM, 20e6, 1500, (40, 40, 6), (25 * MM, 25 * MM), (5 * MM, 9 * MM),
           f_number=0.5), True, 0),
    (_desc(24, 24, 1.6 * MM, 40e6, 2600, (33, 32, 5), (19 * MM, 19 * MM), (5 * MM, 8 * MM),
           f_number=0.5), False, 1),
    # tables of a long receive aperture
    (_desc(16, 1024, 0.1 * MM, 30e6, 400, (33, 64, 7), (1.6 * MM, 3.2 * MM), (4 * MM, 5 * MM)),
     False, 0),
    (_desc(12, 900, 0.1 * MM, 20e6, 300, (40, 33, 4), (2 * MM, 2 * MM), (4 * MM, 5 * MM),
           interp="linear", focal_depth=-8 * MM), False, 2),
])
def test_lds_kernel_with_the_copies_that_fit(dev, desc, iq, most):
    import torch
    desc = dict(desc, iq=iq)
    shape = (desc["n_tx"], desc["n_ch"], desc["n_samples"]) + ((2,) if iq else ())
    e = np.random.default_rng(1).standard_normal(shape).astype(np.float32)
    plan = bfm.Plan(desc, None)
    assert plan.info()["variant"] != 1
    got = plan.das(torch.from_numpy(e).cuda()).cpu().numpy()
    ref = oracle.das_iq(desc, e[..., 0] + 1j * e[..., 1]) if iq else oracle.das(desc, e)
    assert rel_l2(got, ref) <= 1e-5
    axes = _lib.lib().bf_test_set_mirrors(plan._h, 3)
    assert bin(axes).count("1") <= most
