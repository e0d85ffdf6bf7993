"""Small and ragged separable grids (GPU): launches of at most one workgroup
per CU, whose batches may fill a CU's LDS, and odd channel counts split over
groups.

The batch size sets how many windows are staged at once, not the order in
which a point's terms are added (row chunk, then transmit), so every nb must
give the same bits; the image is held to the DAS tests' 1e-5 relative L2
against the FP64 oracle.
"""
import numpy as np
import pytest

import oracle
import paper_2512_11086_amd as bfm
from synth.configs import MM, describe
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu


def _case(mode, n_tx, n_ch, dims, interp, zmax, S=900):
    extra = dict(tx_angles=np.deg2rad(np.linspace(-10, 10, n_tx))) if mode == "tpw" else {}
    if mode == "vls":
        extra["focal_depth"] = -5 * MM
    n_el = max(n_tx, n_ch)
    half = 0.12 * MM * n_el
    y = 0.0 if mode == "forces" else half
    return describe(mode, (n_el, n_el), (0.24 * MM, 0.24 * MM), n_tx, n_ch, S, 20e6, 5e6, dims,
                    (-half, -y, 2 * MM), (half, y, zmax * MM), interp=interp, t0=0.3e-6,
                    f_number=1.0, **extra)


@pytest.mark.parametrize("mode, n_tx, n_ch, dims, interp, zmax, lds", [
    ("forces", 32, 32, (97, 1, 120), "cubic", 22, True),     # one workgroup per CU, ragged boxes
    ("forces", 16, 31, (33, 1, 64), "linear", 22, True),     # channels not a multiple of the row chunk
    ("forces", 12, 5, (16, 1, 9), "cubic", 22, False),       # depth steps too long for the windows
    ("forces", 12, 5, (16, 1, 9), "cubic", 4, True),         # one chunk and a remainder
    ("forces", 8, 8, (5, 1, 3), "cubic", 2.5, False),        # lateral steps too long for them
    ("tpw", 16, 30, (13, 11, 40), "cubic", 12, None),        # either kernel
    ("vls", 16, 16, (17, 5, 33), "linear", 10, None),
])
def test_batch_size_leaves_small_grids_unchanged(mode, n_tx, n_ch, dims, interp, zmax, lds):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = _case(mode, n_tx, n_ch, dims, interp, zmax)
    e = np.random.default_rng(4).standard_normal((n_tx, n_ch, 900)).astype(np.float32)
    e_d = torch.from_numpy(e).cuda()
    plan = bfm.Plan(d, None)
    info = plan.info()
    assert lds is None or (info["variant"] != 1) == lds
    want = plan.das(e_d)
    for nb in (4, 8, 32, 64):
        plan.set_das_config("lds", info["block"], nb)
        now = plan.info()
        assert now["channel_groups"] == info["channel_groups"]
        assert torch.equal(plan.das(e_d), want), (nb, now["nb"])
    assert rel_l2(want.cpu().numpy(), oracle.das(d, e.astype(np.float64))) <= 1e-5
