"""Memory of the partial images of channel-split launches: bf_das_noalloc's static
array holds 8 MiB (larger partial images stay in the plan's own memory, with the
same result), and a frame of a batch holds none while it runs in a persistent
launch."""
import ctypes

import numpy as np
import pytest

import paper_2512_11086_amd as bfm
from paper_2512_11086_amd import _lib
from synth.configs import MM, describe

pytestmark = pytest.mark.gpu


def _volume(dims, n=16, iq=False, S=500):
    half = 0.1 * MM * n
    d = describe("hercules", (n, n), (0.2 * MM, 0.2 * MM), n, n, S, 20e6, 5e6, dims,
                 (-half, -half, 3 * MM), (half, half, 14 * MM), t0=0.5e-6, f_number=1.0)
    if iq:
        d.update(iq=True, fs=10e6)
    return d


def _workspace(plan):
    info = _lib.PlanInfo()
    _lib.check(_lib.lib().bf_plan_get_info(plan._h, ctypes.byref(info)))
    return info.workspace_bytes


def test_noalloc_with_large_partial_images(dev):
    import torch
    d = _volume((64, 64, 128), n=64, iq=True, S=300)
    plan = bfm.Plan(d, None)
    assert plan.info()["channel_groups"] * plan.info()["out_elems"] * 4 > 8 << 20
    e = torch.randn(plan.e_shape, device="cuda")
    want = plan.das(e)
    got = torch.empty_like(want)
    for c in (d["c"], 1.01 * d["c"]):
        _lib.check(_lib.lib().bf_das_noalloc(
            plan._h, ctypes.c_void_p(e.data_ptr()), ctypes.c_void_p(got.data_ptr()), c,
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
        assert torch.equal(got, plan.das(e, c=c))


def test_persistent_frames_hold_no_partial_images(dev):
    import torch
    d = _volume((32, 32, 24))
    one = bfm.Plan(d, None)
    info = one.info()
    part = info["channel_groups"] * info["out_elems"] * 4
    assert info["channel_groups"] > 1
    n = 4
    batch = bfm.BatchPlan([d] * n, [None] * n)
    assert _workspace(batch) == n * info["workspace_bytes"] - (n - 1) * part
    rng = np.random.default_rng(1)
    rfs = [torch.from_numpy(rng.integers(-3000, 3000, (16, 16, 500)).astype(np.int16)).cuda()
           for _ in range(n)]
    outs = [torch.empty(s, device="cuda") for s in batch.out_shapes]
    batch.run(rfs, outs)
    paths = [batch.frame_info(f)["das_path"] for f in range(n)]
    for o, rf in zip(outs, rfs):
        ref = one.das(one.decode(rf)).double()
        assert float((o.double() - ref).norm() / ref.norm()) <= 1e-6
    own = sum(p != "persistent_lds" for p in paths[1:])
    e_bytes = n * 16 * 16 * 500 * 4
    assert _workspace(batch) <= n * info["workspace_bytes"] - (n - 1 - own) * part + e_bytes
