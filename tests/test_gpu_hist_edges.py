"""The energy-angle histogram's bins near their edges, where the float estimate
may not decide, and at magnitudes outside its range: momenta whose energy or
angle is an edge's times 1 + d, d from 0 to 1e-3, zeros, denormals, huge values
and infinities.  Counts and tallies are exact against the definition in double
with the device's own log10, atan2 and sqrt."""
import numpy as np
import pytest

from gpu_common import require_gpu

pytestmark = pytest.mark.gpu

MEC2 = 0.51099895
OFFSETS = [0.0] + [s * d for d in (1e-16, 1e-12, 1e-9, 1e-7, 1e-6, 3e-6, 1e-5, 1e-3) for s in (-1, 1)]
ODD = [0.0, -0.0, 5e-324, 1e-310, 1e-160, 1e-39, 1e-20, 1e-15, 1e-10, 1e10, 1e19, 1e40, 1e160, 1e300,
       np.inf]


def _draw(nE, nA, lo, hi):
    rng = np.random.default_rng(nE * nA)
    d = np.array(OFFSETS)
    K = 10.0 ** (lo + (hi - lo) / nE * np.arange(-1, nE + 2))
    K = (K[:, None] * (1 + d)).ravel()
    K = K[rng.permutation(len(K))]
    th = (np.pi / nA * np.arange(0, nA + 1)[:, None] * (1 + d)).ravel()
    th = np.concatenate([th, rng.uniform(0, np.pi, len(K))])
    K = np.concatenate([rng.choice(K, len(th) - len(K)), K])
    u = np.sqrt(K / MEC2 * (K / MEC2 + 2))
    # the azimuth's edges are the polar angle's shifted, twice as wide
    az = rng.permutation(2 * th - np.pi)
    edge = np.stack([u * np.sin(th) * np.cos(az), u * np.sin(th) * np.sin(az), u * np.cos(th)], 1)
    odd = np.array(ODD + [-v for v in ODD])
    odd = np.stack(np.meshgrid(odd, odd, odd), -1).reshape(-1, 3)
    return np.concatenate([edge, odd])


def _defined(torch, u, nE, nA, lo, hi, angle):
    # divisors as tensors: torch takes a number's reciprocal and multiplies
    def c(v):
        return torch.full((1,), v, dtype=torch.float64, device="cuda")
    x, y, z = u
    up2 = x * x + y * y
    u2 = up2 + z * z
    K = MEC2 * u2 / (torch.sqrt(1.0 + u2) + 1.0)
    fe = torch.floor((torch.log10(K) - lo) / c((hi - lo) / nE))
    a = torch.atan2(torch.sqrt(up2), z) / c(np.pi) if angle == 0 else \
        (torch.atan2(y, x) + np.pi) / c(2.0 * np.pi)
    ia = torch.clamp(torch.floor(a * float(nA)), 0, nA - 1).long()
    fwd = z > 0
    below, above = ~(fe >= 0), fe >= nE
    ok = ~(below | above)
    key = (((~fwd).long() * nE + torch.where(ok, fe, 0.0).long()) * nA + ia)[ok]
    counts = torch.bincount(key, minlength=2 * nE * nA).reshape(2, nE, nA)
    return counts, [int(v.sum()) for v in (fwd, ~fwd, below, above)]


@pytest.mark.parametrize("angle", [0, 1])
@pytest.mark.parametrize("nE,nA,lo,hi", [(1, 1, -3.0, 3.0), (7, 5, -2.0, 2.0), (256, 180, -3.0, 4.0),
                                         (3, 4096, -6.0, 1.0), (5000, 2, -12.0, 12.0)])
def test_bins_at_edges(nE, nA, lo, hi, angle):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    u = [torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in _draw(nE, nA, lo, hi).T]
    c, t = B.rpdla_histogram(torch.zeros_like(u[0]), *u, B.rpdla_hist_spec(nE, nA, lo, hi, angle))
    oc, ot = _defined(torch, u, nE, nA, lo, hi, angle)
    assert torch.equal(c, oc)
    assert t.tolist() == ot + [0, 0]
