"""The energy-angle histogram with energy axes so wide that the distance from
the lower end rounds by more than a float estimate's error: whole counts against
the definition in double, for electrons about an edge that lies among them."""
import numpy as np
import pytest

from gpu_common import require_gpu
from test_gpu_hist_edges import MEC2, _defined

pytestmark = pytest.mark.gpu

# bins, lower and upper end of the axis, the edge [log10 MeV]
AXES = [(1063, -14606963403827.059, 27534332521.8125, -1.8905321841911231),
        (51915013, -10928177843366.89, 10773519584765.668, 1.2859060994196172),
        (17, -21885146179564.945, 24620789452016.03, 2.5755753759489464),
        (2, -1.0e6, 1.0e6, 0.0), (40, -1.1e6, 3.3e6, 0.0)]


@pytest.mark.parametrize("nE,lo,hi,edge", AXES)
@pytest.mark.parametrize("angle", [0, 1])
def test_wide_axis(nE, lo, hi, edge, angle):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    n = 4096
    rng = np.random.default_rng(nE)
    lk = edge + rng.uniform(-1, 1, n) * np.where(np.arange(n) % 2 == 0, 1e-3, 4e-16 * abs(lo))
    K = 10.0 ** np.clip(lk, -6, 6)
    u = np.sqrt(K / MEC2 * (K / MEC2 + 2))
    th, az = rng.uniform(0, np.pi, n), rng.uniform(-np.pi, np.pi, n)
    m = [torch.as_tensor(v, device="cuda") for v in
         (u * np.sin(th) * np.cos(az), u * np.sin(th) * np.sin(az), u * np.cos(th))]
    print(f"wide axis: {nE} bins of {lo} .. {hi}", flush=True)
    c, t = B.rpdla_histogram(torch.zeros_like(m[0]), *m, B.rpdla_hist_spec(nE, 2, lo, hi, angle))
    oc, ot = _defined(torch, m, nE, 2, lo, hi, angle)
    assert torch.equal(c, oc)
    assert t.tolist() == ot + [0, 0]
