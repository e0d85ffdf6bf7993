"""A column with an infinite or NaN sample has a non-finite envelope at every
depth (each output of the Hilbert transform sums over the whole column, and
the zeros of its kernel are no reason to leave a sample out); the other columns
are the envelope they are without it, bit for bit."""
import pytest

import paper_2512_11086_amd as bfm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(20, 96), (5, 250), (18, 101), (4100, 48), (17, 22), (40, 1000)])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_nonfinite_column(dev, shape, bad):
    import torch
    x = torch.randn(shape, generator=torch.Generator().manual_seed(3)).cuda()
    env = bfm.Envelope(shape)
    want = env(x)
    for col, at in ((2, 7), (shape[0] - 1, shape[1] - 2)):
        y = x.clone()
        y[col, at] = bad
        got = env(y)
        assert not torch.isfinite(got[col]).any()
        keep = torch.arange(shape[0]) != col
        assert torch.equal(got[keep], want[keep])
