"""The ionization kernel at the edges of its split (one wave per atom, 64
panels at a time, four waves a block): windows of fewer, exactly and just over
64 panels, atom counts around a block's four, one and ten states, steps much
coarser and finer than the default, against the oracle on the same atoms.

Tolerance: birth times to 1e-10 max(|t|, T), the rule of the other
ionization tests; the same born / unborn pattern.
"""
import numpy as np
import pytest

import seeded_inputs as SI
from gpu_common import BEAM, C_LIGHT, require_gpu

pytestmark = pytest.mark.gpu

# atoms, first and last state, panels before and after the peak, steps per period
CASES = [
    (1, 1, 1, None, None, 200),
    (3, 1, 10, None, None, 200),
    (4, 8, 8, 31, 1, 200),        # 32 panels: half a wave
    (5, 1, 6, 63, 1, 200),        # exactly 64
    (6, 1, 6, 64, 1, 200),        # one past
    (7, 1, 10, 500, 141, 200),    # 641: ten waves of panels and one panel
    (9, 1, 10, None, None, 16),   # coarse steps: several births in one panel
    (2, 5, 9, None, None, 1000),  # fine steps
]


@pytest.mark.parametrize("n,kf,kl,before,after,per", CASES)
@pytest.mark.parametrize("window", [0, 1])
def test_ionize_edges(orc, n, kf, kl, before, after, per, window):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    T = BEAM["lam"] / C_LIGHT
    dt = T / per
    kw = dict(dt=dt, window=window)
    if before is not None:
        kw.update(t_before=before * dt, t_after=after * dt)
    L = B.rpdla_laser_init_intensity(BEAM["lam"], BEAM["w0"], BEAM["tau"], BEAM["I"], **kw)
    OL = orc.laser_intensity(BEAM["lam"], BEAM["w0"], BEAM["tau"], BEAM["I"])
    for k, v in kw.items():
        orc._set(OL, k, v)
    xs, ys, zs = SI.cylinder_atoms(100 + n, n, BEAM["w0"], 2e-6)
    x, y, z = (torch.as_tensor(a, device="cuda") for a in (xs, ys, zs))
    K = kl - kf + 1
    print(f"ionize {n} atoms, states {kf}-{kl}, {per} steps, window {window}", flush=True)
    tb = torch.full((n * K + 8,), -7.0, dtype=torch.float64, device="cuda")
    B.rpdla_ionize(L, 11, 2, 5, x, y, z, kf, kl, tb)
    g = tb.cpu().numpy()
    assert np.all(g[n * K:] == -7.0)               # nothing past the last slot
    g = g[:n * K]
    o = orc.ionize(OL, 11, 2, 5, xs, ys, zs, kf, kl)
    fin = np.isfinite(o)
    assert fin.any()
    assert np.array_equal(fin, np.isfinite(g)) and np.all(np.isposinf(g[~fin]))
    assert np.all(np.abs(g[fin] - o[fin]) <= 1e-10 * np.maximum(np.abs(o[fin]), T))
