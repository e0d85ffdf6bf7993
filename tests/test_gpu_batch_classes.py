"""Small HERCULES frames of a batch, one with a symmetric aperture and one without,
run as one kernel class: mirror points for the one alone would split them into
launches that follow each other."""
import numpy as np
import pytest

import oracle
import paper_2512_11086_amd as bfm
from synth.configs import MM, describe
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu


def _frame(tx, cols=32, dims=(31, 31, 40), S=500):
    half = 0.1 * MM * cols
    n_tx = len(tx)
    return describe("hercules", (cols, cols), (0.2 * MM, 0.2 * MM), n_tx, 30, S, 20e6, 5e6, dims,
                    (-half, -half, 3 * MM), (half, half, 14 * MM), t0=0.5e-6, f_number=1.0,
                    tx_elements=tx, channel_map=np.arange(30) * cols // 30)


def test_small_frames_stay_in_one_class(dev):
    import torch
    descs = [_frame(np.r_[0:2, 30:32]), _frame(np.arange(28)), _frame(np.arange(28))]
    batch = bfm.BatchPlan(descs, [None] * 3)
    rng = np.random.default_rng(4)
    rfs = [torch.from_numpy(rng.integers(-3000, 3000, (d["n_tx"], 30, 500)).astype(np.int16)).cuda()
           for d in descs]
    outs = [torch.empty(s, device="cuda") for s in batch.out_shapes]
    for step in (batch.run, batch.graph_launch, batch.graph_launch):
        for o in outs:
            o.zero_()
        step(rfs, outs)
        for o, d, rf in zip(outs, descs, rfs):
            assert rel_l2(o.cpu().numpy(), oracle.das(d, rf.cpu().numpy().astype(np.float64))) <= 1e-5
    info = [batch.frame_info(f) for f in range(3)]
    assert {i["das_path"] for i in info} == {"persistent_lds"}
    assert len({i["das_class"] for i in info}) == 1
