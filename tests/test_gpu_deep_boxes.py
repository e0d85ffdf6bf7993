"""HERCULES boxes of many depths keep the precision of the default's 6: the rows of
wavefronts of a deep box have delay references of their own.

The error against the FP64 oracle is dominated by the FP32 positions here (steps
of 20 samples and white data).  Emulated position errors (RMS in samples): 1.74e-6
for 6 depths with one reference, 1.48e-6 for 4 depths, 2.2 and 5.1e-6 for 8 and 24
depths with one reference; so a deep box may be at most as far off as the default
one, and 10 % for the rest of the rounding.
"""
import numpy as np
import pytest

import oracle
import paper_2512_11086_amd as bfm
from paper_2512_11086_amd import _lib
from synth.configs import MM, describe
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("allowed", [0, 3])
@pytest.mark.parametrize("e_type, focal", [("f32", None), ("i32", None), ("f32", -9.0)])
def test_deep_boxes_are_as_precise_as_the_default(dev, allowed, e_type, focal):
    import torch
    n, S, half = 24, 2200, 2.4 * MM
    kw = dict(focal_depth=focal * MM) if focal else {}
    d = describe("hercules", (n, n), (0.2 * MM, 0.2 * MM), n, n, S, 30e6, 7.5e6, (26, 24, 96),
                 (-half, -half, 4 * MM), (half, half, 52 * MM), t0=0.0, f_number=1.0, **kw)
    e = np.rint(np.random.default_rng(6).standard_normal((n, n, S)) * 3000).astype(np.float32)
    t = torch.from_numpy(e).cuda()
    if e_type == "i32":
        t = t.to(torch.int32)
    ref = oracle.das(d, e)

    def error(axes, tile, block):
        plan = bfm.Plan(d, None, e_type=e_type)
        _lib.lib().bf_test_set_mirrors(plan._h, axes)
        plan.set_tile(*tile)
        plan.set_das_config("lds2", block, 48)
        assert plan.info()["variant"] == 2
        return rel_l2(plan.das(t).cpu().numpy(), ref)

    most = 1.1 * error(0, (3, 3, 0), (2, 2, 3))        # 6 depths, one reference
    for tile, block in (((3, 3, 0), (2, 2, 3)), ((2, 3, 1), (3, 2, 2)), ((3, 2, 1), (2, 1, 6)),
                        ((3, 3, 0), (2, 1, 6)), ((2, 3, 1), (1, 1, 12))):
        assert error(allowed, tile, block) <= most, (tile, block)
