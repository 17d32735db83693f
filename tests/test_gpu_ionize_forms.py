"""The ionization's forms give the same bits: calls that the rule takes lane by
lane in the order of the work, or many atoms to a wave, against the same atoms in
calls below 16,384, which take a wave each.  Windows of few and many panels,
lasers that reach no state, a few, one and all, both window kinds, every field
order, one state and ten, sizes around a block and a wave's share; and the order
as a permutation under graph capture and on two streams."""
import numpy as np
import pytest

from gpu_common import require_gpu

pytestmark = pytest.mark.gpu

DT = 0.8e-6 / 299792458.0 / 200
PIECE = 16000
# field, intensity [W/cm^2], window in panels (None: the default), states, atoms, window kind
CASES = [
    (5, 1e14, None, (1, 10), 16384, 0),      # closed: many atoms to a wave
    (5, 1.5e15, None, (1, 10), 70001, 0),    # a few open
    (5, 4e15, None, (1, 3), 200003, 0),
    (5, 1.5e20, None, (9, 10), 65537, 1),
    (5, 1e21, 256, (1, 10), 149201, 0),      # few panels: a lane each
    (5, 1e21, 256, (8, 8), 59201, 1),
    (5, 1e21, 33, (3, 9), 102500, 0),
    (3, 1e21, 300, (1, 2), 72501, 0),
    (1, 5e18, 300, (7, 9), 82501, 0),
    (10, 1e21, 200, (1, 4), 85001, 0),
    (10, 1e14, None, (1, 10), 20000, 0),
    (11, 1e21, 150, (1, 5), 100001, 0),      # uniform field
    (21, 1e21, 200, (1, 4), 85001, 1),
    (23, 1e14, None, (1, 10), 17001, 0),
    (25, 1e21, 200, (1, 4), 85001, 0),
    (25, 1e14, None, (1, 10), 17001, 0),
]


def _laser(B, field, I, panels, kind):
    kw = {} if panels is None else dict(t_before=0.5 * panels * DT, t_after=0.5 * panels * DT)
    L = B.rpdla_laser_init_intensity(0.8e-6, 3e-6, 30e-15, I, window=kind, **kw)
    L.field = field
    if field == 11:
        L.test_E[0], L.test_E[2] = 2e11, 3e11
    return L


def _pieces(torch, B, L, seed, x, y, z, kf, kl):
    return torch.cat([B.rpdla_ionize(L, seed, 3, a, x[a:a + PIECE].contiguous(),
                                     y[a:a + PIECE].contiguous(), z[a:a + PIECE].contiguous(), kf, kl)
                      for a in range(0, x.numel(), PIECE)])


@pytest.mark.parametrize("field,I,panels,states,n,kind", CASES)
def test_forms_agree(field, I, panels, states, n, kind):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    L = _laser(B, field, I, panels, kind)
    kf, kl = states
    x, y, z = B.rpdla_sample_atoms(7, 3, 0, n, 2 * L.w0, B.rpdla_rayleigh(L))
    odd = torch.tensor([float("nan"), float("inf"), 0.0, -float("inf")], dtype=torch.float64, device="cuda")
    x[5:9], z[11:15] = odd, odd
    print(f"ionize field {field} I {I:g} panels {panels} states {states} atoms {n}", flush=True)
    got = torch.full((n * (kl - kf + 1) + 8,), -7.0, dtype=torch.float64, device="cuda")
    B.rpdla_ionize(L, 11, 3, 0, x, y, z, kf, kl, got)
    assert bool((got[-8:] == -7.0).all())
    ref = _pieces(torch, B, L, 11, x, y, z, kf, kl)
    assert torch.equal(got[:-8].view(torch.int64), ref.view(torch.int64))


@pytest.mark.parametrize("I,panels,n", [(1e21, 128, 150001), (1e14, None, 20001)])
def test_capture_and_streams(I, panels, n):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    L = _laser(B, 5, I, panels, 0)
    x, y, z = B.rpdla_sample_atoms(7, 3, 0, n, 2 * L.w0, B.rpdla_rayleigh(L))
    want = [B.rpdla_ionize(L, seed, 3, 0, x, y, z, 1, 10) for seed in (1, 2)]
    out = torch.empty(n * 10, dtype=torch.float64, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        B.rpdla_ionize(L, 1, 3, 0, x, y, z, 1, 10, out)
    for _ in range(4):
        out.fill_(5.0)
        assert float(torch.arange(1000, device="cuda", dtype=torch.float64).sum()) == 499500.0
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int64), want[0].view(torch.int64))
    streams = [torch.cuda.Stream() for _ in range(2)]
    for _ in range(3):
        got = []
        for seed, st in zip((1, 2), streams):
            with torch.cuda.stream(st):
                got.append(B.rpdla_ionize(L, seed, 3, 0, x, y, z, 1, 10))
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.int64), b.view(torch.int64))


@pytest.mark.parametrize("field,I,panels,n_cfg,n,apc", [
    (5, 1e14, None, 3, 6001, 6001),        # no state reached: many atoms to a wave
    (5, 1e14, None, 2, 20000, 9001),       # a partial last chunk
    (5, 1e21, 200, 2, 80001, 80001),       # few panels: a lane per atom
    (25, 1e21, 200, 1, 170000, 150001),
    (11, 1e21, 150, 2, 60000, 60000),      # uniform field
])
def test_sweep_forms_agree(field, I, panels, n_cfg, n, apc):
    """A sweep's births against those of the single calls' wave form, on its last
    chunk, captured and replayed."""
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    kf, kl, seed = 1, 3, 11
    lasers = [_laser(B, field, I, panels, 0) for _ in range(n_cfg)]
    ws = torch.zeros(B.rpdla_batched_workspace_bytes(n_cfg, apc, kf, kl), dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    print(f"sweep field {field} I {I:g} panels {panels}: {n_cfg} x {n} by {apc}", flush=True)
    first = (n - 1) // apc * apc
    for _ in range(2):
        B.rpdla_run_batched(lasers, seed, 40, n, apc, 2.0, kf, kl, 0,
                            B.rpdla_hist_spec(8, 4, -6.0, 3.0, 0), workspace=ws, stream=s)
        s.synchronize()
        a = B.batched_chunk_arrays(ws, n_cfg, apc, kf, kl)
        for c in range(n_cfg):
            m = n - first
            x, y, z = (a[k][c, :m].contiguous() for k in ("x", "y", "z"))
            ref = torch.cat([B.rpdla_ionize(lasers[c], seed, 40 + c, first + i, x[i:i + PIECE].contiguous(),
                                            y[i:i + PIECE].contiguous(), z[i:i + PIECE].contiguous(), kf, kl)
                             for i in range(0, m, PIECE)])
            got = a["t_birth"][c, :m].reshape(-1).contiguous()
            assert torch.equal(got.view(torch.int64), ref.view(torch.int64))
