"""Planes of IQ, BF16 and INT32 data whose channel sum is split over groups
(odd channel counts, more groups than 16 among them) against the FP64 oracle.

Tolerance: the DAS tests' 1e-5 relative L2.  A split changes the order of the
channel sum alone, so the noalloc entry point, which runs the same launch, gives
the same bits.
"""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2512_11086_amd as bfm
from paper_2512_11086_amd import _lib
from synth.configs import MM, describe
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["iq", "bf16", "i32"])
@pytest.mark.parametrize("n_tx, n_ch, dims, interp, many", [
    (12, 42, (60, 1, 60), "cubic", 11),
    (8, 128, (65, 1, 40), "linear", 8),
    (5, 31, (33, 1, 70), "cubic", 3),
    (16, 3, (20, 1, 17), "linear", 1),
    (24, 102, (64, 1, 33), "cubic", 17),
])
def test_split_planes_match_oracle(dev, kind, n_tx, n_ch, dims, interp, many):
    import torch
    n_el, S = 128, 600
    half = 0.05 * MM * n_el
    d = describe("forces", (n_el, n_el), (0.1 * MM, 0.1 * MM), n_tx, n_ch, S, 20e6, 5e6, dims,
                 (-half, 0.0, 4 * MM), (half, 0.0, 12 * MM), interp=interp, t0=0.2e-6, f_number=1.0)
    d.update(iq=kind == "iq", fs=8e6 if kind == "iq" else 20e6)
    shape = (n_tx, n_ch, S) + ((2,) if d["iq"] else ())
    e = np.rint(np.random.default_rng(n_ch).standard_normal(shape) * 1000).astype(np.float32)
    t = torch.from_numpy(e).cuda()
    if kind != "iq":
        t = t.to(torch.bfloat16 if kind == "bf16" else torch.int32)
        e = t.to(torch.float32).cpu().numpy()
    plan = bfm.Plan(d, None, e_type="f32" if kind == "iq" else kind)
    assert plan.info()["channel_groups"] >= many
    got = plan.das(t)
    ref = oracle.das_iq(d, e[..., 0] + 1j * e[..., 1]) if d["iq"] else oracle.das(d, e)
    assert rel_l2(got.cpu().numpy(), ref) <= 1e-5
    again = torch.empty_like(got)
    _lib.check(_lib.lib().bf_das_noalloc(plan._h, ctypes.c_void_p(t.data_ptr()),
                                         ctypes.c_void_p(again.data_ptr()), d["c"],
                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    assert torch.equal(again, got)
