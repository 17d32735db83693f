"""Which form a push takes changes no bits.  Calls on both sides of the rule
that leaves a push of few steps to the queue, at every field order and form,
against the other form (small calls are ordered, rpdla_push_noalloc is the
queue); time-sliced ordered pushes at the orders and forms that the other tests
do not slice; a push under graph capture, replayed with other work between; and
pushes on two streams at once."""
import numpy as np
import pytest

import seeded_inputs as SI
from gpu_common import require_gpu

pytestmark = pytest.mark.gpu

PIECE = 65536          # one wave per SIMD on 256 CUs: no slices
DT = 0.8e-6 / 299792458.0 / 200


def _case(torch, B, n, K, field, steps, spread, seed):
    L = B.rpdla_laser_init_intensity(0.8e-6, 2e-6, 4e-15, 1e21, t_before=0.5 * steps * DT,
                                     t_after=0.5 * steps * DT)
    L.field = field
    if field == 11:
        L.test_E[0], L.test_E[2], L.test_B[1] = 3e11, 1e12, 1e3
    xs, ys, zs = SI.cylinder_atoms(seed, n, 4e-6, 10e-6)
    rng = np.random.default_rng([n, K, seed])
    tb = (zs[:, None] / 299792458.0 + spread * steps * DT * rng.uniform(-0.5, 0.5, (n, K))).ravel()
    tb[rng.uniform(size=n * K) < 0.07] = np.inf
    tb[:4] = np.nan, -1.0, 1.0, -np.inf
    return L, [torch.as_tensor(a, device="cuda") for a in (tb, xs, ys, zs)]


def _push(B, form, L, tb, xyz, K):
    if form == "rr":
        return B.rpdla_push_rr(L, 1, tb, *xyz, K)
    return B.rpdla_push(L, B.RPDLA_MIXED if form == "mixed" else B.RPDLA_FP64, tb, *xyz, K)


def _other(torch, B, form, L, tb, xyz, K):
    """The same slots through calls of a single slice, all ordered."""
    step = PIECE // K * K
    parts = [_push(B, form, L, tb[a:a + step].contiguous(),
                   [v[a // K:(a + step) // K].contiguous() for v in xyz], K)
             for a in range(0, tb.numel(), step)]
    return [torch.cat(p) for p in zip(*parts)]


def _same(got, ref):
    for g, r in zip(got, ref):
        g, r = g.cpu().numpy(), r.cpu().numpy()
        nan = np.isnan(r)
        assert np.array_equal(nan, np.isnan(g))
        assert np.array_equal(g[~nan].view(np.uint64), r[~nan].view(np.uint64))


FORMS = [("fp64", f) for f in (1, 3, 5, 10, 11, 21, 23, 25)] + \
        [("mixed", f) for f in (1, 3, 5, 10, 11)] + [("rr", f) for f in (1, 3, 5, 10, 11, 21, 23, 25)]


@pytest.mark.parametrize("form,field", FORMS)
def test_few_steps(form, field):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    # the last size below the rule, the first of it, and some with one step too many
    for n, steps in ((2**16, 4), (2**16 + 1, 4), (70001, 5), (2**18 + 7, 3), (2**18 + 65, 4)):
        print(f"{form} field {field}: {n} slots of {steps} steps", flush=True)
        L, (tb, *xyz) = _case(torch, B, n, 1, field, steps, 1.0, 1)
        _same(_push(B, form, L, tb, xyz, 1), _other(torch, B, form, L, tb, xyz, 1))


@pytest.mark.parametrize("form,field", FORMS)
def test_slices(form, field):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    n, K = 36001, 3                   # 1.6 waves per SIMD on 256 CUs
    print(f"{form} field {field}: {n} x {K} slots in slices", flush=True)
    L, (tb, *xyz) = _case(torch, B, n, K, field, 300, 0.9, 2)
    got = _push(B, form, L, tb, xyz, K)
    if form == "rr":
        _same(got, _other(torch, B, form, L, tb, xyz, K))
    else:
        _same(got, B.rpdla_push_noalloc(L, B.RPDLA_MIXED if form == "mixed" else B.RPDLA_FP64, tb,
                                        *xyz, K, tuple(torch.empty_like(tb) for _ in range(6))))


@pytest.mark.parametrize("form", ["fp64", "mixed", "rr"])
@pytest.mark.parametrize("n,steps", [(500, 200), (70001, 200), (2**18 + 1, 2)])
def test_capture(form, n, steps):
    """One slice, several, and the queue."""
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    L, (tb, *xyz) = _case(torch, B, n, 1, 5, steps, 0.9, 3)
    _, (tb2, *xyz2) = _case(torch, B, n, 1, 5, steps, 0.9, 4)
    want = [_push(B, form, L, t, p, 1) for t, p in ((tb, xyz), (tb2, xyz2))]
    bufs = [torch.empty_like(v) for v in (tb, *xyz)]
    out = tuple(torch.empty_like(tb) for _ in range(6))
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    print(f"capture {form}: {n} slots of {steps} steps", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        if form == "rr":
            B.rpdla_push_rr(L, 1, *bufs, 1, out=out, want_chi=False)
        else:
            B.rpdla_push(L, B.RPDLA_MIXED if form == "mixed" else B.RPDLA_FP64, *bufs, 1, out)
    for rep in range(4):
        for b, v in zip(bufs, (tb, *xyz) if rep % 2 == 0 else (tb2, *xyz2)):
            b.copy_(v)
        for o in out:
            o.fill_(5.0)
        assert float(torch.arange(1000, device="cuda", dtype=torch.float64).sum()) == 499500.0
        g.replay()
        torch.cuda.synchronize()
        _same(out, want[rep % 2][:6])


@pytest.mark.parametrize("form", ["fp64", "mixed", "rr"])
def test_two_streams(form):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    cases = [_case(torch, B, 40000 + 30000 * i, 2, 5, 250, 0.9, 5 + i) for i in range(2)]
    want = [_push(B, form, L, a[0], a[1:], 2) for L, a in cases]
    streams = [torch.cuda.Stream() for _ in cases]
    torch.cuda.synchronize()
    for _ in range(3):
        got = []
        for st, (L, a) in zip(streams, cases):
            with torch.cuda.stream(st):
                got.append(_push(B, form, L, a[0], a[1:], 2))
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            _same(g, w)


@pytest.mark.parametrize("precision,field", [(0, f) for f in (1, 3, 10, 11, 21, 23, 25)] +
                         [(1, f) for f in (1, 3, 10, 11)])
def test_sweep_forms(precision, field):
    """A sweep's ordered push against its queue at the other field orders:
    births, momenta, counts, tallies and steps."""
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    n_cfg, n, kf, kl = 2, 4500, 1, 10
    lasers = []
    for c in range(n_cfg):
        L = B.rpdla_laser_init_intensity((0.8 + 0.2 * c) * 1e-6, 2e-6, 4e-15, 1e21,
                                         t_before=(150 + 40 * c) * DT, t_after=150 * DT)
        L.field = field
        if field == 11:
            L.test_E[0], L.test_E[2], L.test_B[1] = 3e11, 1e12, 1e3
        lasers.append(L)
    lay = B.rpdla_batched_workspace_layout(n_cfg, n, kf, kl)
    chunk = lay["uz"] + (n_cfg * n * 10 * 8 + 255) // 256 * 256
    got = []
    print(f"sweep field {field} precision {precision}", flush=True)
    for size in (B.rpdla_batched_workspace_bytes(n_cfg, n, kf, kl), chunk):
        ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
        steps = torch.zeros(n_cfg, dtype=torch.int64, device="cuda")
        c, t = B.rpdla_run_batched(lasers, 5, 40, n, n, 2.0, kf, kl, precision,
                                   B.rpdla_hist_spec(32, 18, -6.0, 3.0, 0), workspace=ws,
                                   electron_steps=steps)
        a = B.batched_chunk_arrays(ws, n_cfg, n, kf, kl)
        born = torch.isfinite(a["t_birth"])
        zero = torch.zeros((), dtype=torch.float64, device="cuda")
        got.append([c, t, steps, a["t_birth"].clone()] +
                   [torch.where(born, a[k], zero) for k in ("ux", "uy", "uz")])
    for x, y in zip(*got):
        assert torch.equal(x.contiguous().view(torch.int64), y.contiguous().view(torch.int64))
    assert int(got[0][2].sum()) > 0
