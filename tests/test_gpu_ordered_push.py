"""The ordered push (slots sorted by step count, dealt to waves in rounds and
time slices) against the queue push of the same slots (rpdla_push_noalloc; with
radiation reaction, which has no such form, against calls of at most 65,536
slots, which need no slices on 256 CUs): bitwise the same outputs, for slot counts
around whole groups of 64, one group per SIMD and two, with few or no born slots,
and with births outside the window, on step counts from one to a few hundred."""
import numpy as np
import pytest

import seeded_inputs as SI
from gpu_common import require_gpu

pytestmark = pytest.mark.gpu

PIECE = 65536
# atoms, slots per atom, fraction born
CASES = [(1, 1, 1.0), (63, 1, 1.0), (13, 5, 1.0), (65, 1, 0.9), (1000, 3, 0.8), (65537, 1, 0.9), (65600, 1, 1.0), (131136, 1, 1.0), (66666, 3, 0.8), (30011, 10, 0.9),
         (70000, 1, 0.01), (65537, 1, 0.0)]


def _case(torch, B, n, K, born, order):
    L = B.rpdla_laser_init_intensity(0.8e-6, 2e-6, 2e-15, 1e21)
    L.field = order
    xs, ys, zs = SI.cylinder_atoms(n + K, n, 4e-6, 10e-6)
    rng = np.random.default_rng([n, K])
    tb = (zs[:, None] / 299792458.0 + 2e-15 * rng.normal(size=(n, K))).ravel()
    tb[rng.uniform(size=n * K) >= born] = np.inf
    if born > 0 and n * K > 64:
        tb[3], tb[4], tb[5], tb[6] = np.nan, -1.0, 1.0, -np.inf      # outside the window
    return L, [torch.as_tensor(a, device="cuda") for a in (tb, xs, ys, zs)]


def _pieces(torch, push, tb, xyz, K):
    step = PIECE // K * K
    parts = [push(tb[a:a + step].contiguous(), [v[a // K:a // K + step // K].contiguous()
                                                for v in xyz])
             for a in range(0, tb.numel(), step)]
    return [torch.cat(p) for p in zip(*parts)]


@pytest.mark.parametrize("n,K,born", CASES)
@pytest.mark.parametrize("form,order", [("fp64", 5), ("mixed", 5), ("rr", 1)])
def test_ordered_push_equals_queue_push(n, K, born, form, order):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    L, (tb, *xyz) = _case(torch, B, n, K, born, order)

    def push(t, pos):
        if form == "rr":
            return B.rpdla_push_rr(L, 1, t, *pos, K)
        return B.rpdla_push(L, B.RPDLA_MIXED if form == "mixed" else B.RPDLA_FP64, t, *pos, K)

    print(f"ordered push {form}: {n} x {K} slots, {born} born", flush=True)
    for _ in range(2):
        got = push(tb, xyz)
    if form == "rr":
        ref = _pieces(torch, push, tb, xyz, K)
    else:
        ref = B.rpdla_push_noalloc(L, B.RPDLA_MIXED if form == "mixed" else B.RPDLA_FP64, tb, *xyz,
                                   K, tuple(torch.empty_like(tb) for _ in range(6)))
    for g, r in zip(got, ref):
        g, r = g.cpu().numpy(), r.cpu().numpy()
        nan = np.isnan(r)
        assert np.array_equal(nan, np.isnan(g))
        assert np.array_equal(g[~nan].view(np.uint64), r[~nan].view(np.uint64))
    assert born == 0.0 or np.isfinite(got[0].cpu().numpy()).sum() >= born * n * K * 0.9
