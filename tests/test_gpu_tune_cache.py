"""The tuning cache tells plans with mirror points from plans without (their
launches differ in points per lane, batch and LDS layout), and an entry that
would take a plan off the LDS kernel is not applied."""
import numpy as np
import pytest

import oracle
import paper_2512_11086_amd as bfm
from synth.configs import MM, describe
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu


def _desc(**kw):
    n, half = 16, 1.6 * MM
    return describe("hercules", (n, n), (0.2 * MM, 0.2 * MM), n, n, 500, 20e6, 5e6, (33, 32, 24),
                    (-half, -half, 3 * MM), (half, half, 12 * MM), t0=0.5e-6, f_number=1.0, **kw)


def test_mirrored_and_plain_plans_have_their_own_entries(dev, tmp_path):
    cache = str(tmp_path / "tune.txt")
    keys = []
    for kw in ({}, dict(channel_map=np.roll(np.arange(16), 1)),
               dict(channel_map=np.roll(np.arange(16), 1), tx_elements=np.roll(np.arange(16), 1))):
        bfm.Plan(_desc(**kw), None).autotune(cache)
        keys = [ln.split()[0] for ln in open(cache).read().splitlines()]
    assert len(set(keys)) == 3
    assert [k.endswith(m) for k, m in zip(keys, ("|mir3", "|mir2", "|et0"))] == [True] * 3


def test_entry_that_does_not_fit_is_left_out(dev, tmp_path):
    import torch
    cache = str(tmp_path / "tune.txt")
    d = _desc()
    plan = bfm.Plan(d, None)
    before = plan.info()
    assert before["variant"] != 1
    plan.autotune(cache)
    key = open(cache).read().split()[0]
    with open(cache, "w") as f:      # 64 depths per wavefront, 16 wavefronts deep: no such window fits
        f.write(f"{key} 0 0 6 1 1 16 48 2\n")
    fresh = bfm.Plan(d, None)
    now = fresh.autotune(cache)
    assert (now["variant"], now["tile"], now["block"]) == \
        (before["variant"], before["tile"], before["block"])
    e = np.random.default_rng(0).standard_normal((16, 16, 500)).astype(np.float32)
    assert rel_l2(fresh.das(torch.from_numpy(e).cuda()).cpu().numpy(), oracle.das(d, e)) <= 1e-5
