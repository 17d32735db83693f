"""The histograms on both sides of their rule (bins in a block's LDS up to 8192,
a table of 16,384 places in LDS beyond), for slot counts around a wave and a block and past
one pass of the whole grid, with bins that many slots share, against the
oracle's binning of the same numbers: counts and tallies exact."""
import numpy as np
import pytest

from gpu_common import require_gpu

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (64, 64), (4097, 1), (64, 65), (256, 180),
          (16385, 2)]     # 2, 8192, 8194, 8320, 92160 and 65540 bins
SIZES = [1, 63, 64, 65, 1023, 1024, 1025, 3000]


def _t(torch, a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def _draw(n):
    rng = np.random.default_rng(n)
    u = rng.normal(size=(n, 3)) * np.exp(rng.uniform(-3, 5, size=(n, 1)))
    u[::3] = u[0]                                # one crowded bin
    tb = np.where(rng.uniform(size=n) < 0.1, np.inf, 0.0)
    u[rng.uniform(size=n) < 0.02, 1] = np.nan
    return tb, u


@pytest.mark.parametrize("nE,nA", SHAPES)
@pytest.mark.parametrize("n,times", [(n, 1) for n in SIZES] + [(3000, 200)])
def test_histograms_exact(orc, nE, nA, n, times):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    tb, u = _draw(n)
    big = [_t(torch, np.tile(a, times)) for a in (tb, u[:, 0], u[:, 1], u[:, 2])]
    c, t = B.rpdla_histogram(*big, B.rpdla_hist_spec(nE, nA, -3.0, 3.0, 0))
    oc, ot = orc.histogram(tb, u[:, 0], u[:, 1], u[:, 2], nE, nA, -3.0, 3.0, 0)
    assert np.array_equal(c.cpu().numpy().astype(np.uint64), times * oc)
    assert np.array_equal(t.cpu().numpy().astype(np.uint64), times * ot)
    c, t = B.rpdla_histogram2d(*big[1:], B.rpdla_hist2d_spec(nE, nA, -4.0, 4.0, -2.0, 2.0))
    oc, ot = orc.histogram2d(u[:, 0], u[:, 1], u[:, 2], nE, -4.0, 4.0, nA, -2.0, 2.0)
    assert np.array_equal(c.cpu().numpy().astype(np.uint64), times * oc)
    assert np.array_equal(t.cpu().numpy().astype(np.uint64), times * ot)
