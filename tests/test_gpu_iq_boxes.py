"""IQ HERCULES images do not depend on the workgroup's box.

An IQ term's position is its lane's own integer sample plus an FP32 excess and
fraction, so the box a point is computed in (its lane tile, the workgroup's
shape) changes neither a delay nor a phase, and the traces are added in the
same order: boxes of 2 to 24 depths give the same bits, here with depth steps of
9 and 18 samples there and back.  (A position relative to a reference of the box
loses bits of its fraction with the box's depth.)
"""
import numpy as np
import pytest

import oracle
import paper_2512_11086_amd as bfm
from paper_2512_11086_amd import _lib
from synth.configs import MM, describe
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz, focal", [(25, None), (13, None), (13, -9.0)])
@pytest.mark.parametrize("interp", ["cubic", "linear"])
def test_iq_image_is_independent_of_the_box(dev, nz, focal, interp):
    import torch
    n, S = 16, 900
    half = 0.1 * MM * n
    kw = dict(focal_depth=focal * MM) if focal else {}
    d = describe("hercules", (n, n), (0.2 * MM, 0.2 * MM), n, n, S, 15e6, 5e6, (18, 17, nz),
                 (-half, -half, 4 * MM), (half, half, 15 * MM), t0=1e-6, f_number=1.0,
                 interp=interp, **kw)
    d["iq"] = True
    rng = np.random.default_rng(2)
    e = rng.standard_normal((n, n, S, 2)).astype(np.float32)
    e_d = torch.from_numpy(e).cuda()
    plan = bfm.Plan(d, None)
    _lib.lib().bf_test_set_mirrors(plan._h, 0)
    want = None
    for tile, block in (((3, 3, 0), (2, 2, 3)), ((3, 3, 0), (2, 1, 6)), ((2, 3, 1), (2, 2, 3)),
                        ((3, 2, 1), (1, 1, 12)), ((3, 3, 0), (3, 2, 2))):
        plan.set_tile(*tile)
        plan.set_das_config("lds", block, 64)
        assert plan.info()["variant"] == 0
        got = plan.das(e_d)
        if want is None:
            want = got
            ref = oracle.das_iq(d, e[..., 0] + 1j * e[..., 1])
            assert rel_l2(want.cpu().numpy(), ref) <= 1e-5
        assert torch.equal(got, want), (tile, block)
