"""Ordered pushes of so many born slots that groups are pushed in whole rounds
of resident waves before the time slices: just below two rounds, exactly two,
two and a part, and three and a part, bitwise against the queue push (radiation
reaction: against ordered calls of one slice), in windows of a few dozen steps;
and a batched sweep of as many against its queue."""
import ctypes as C

import numpy as np
import pytest

from gpu_common import require_gpu
from test_gpu_push_routes import DT, _other, _push, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,field", [("fp64", 5), ("mixed", 5), ("rr", 5), ("fp64", 21),
                                        ("fp64", 25), ("mixed", 10), ("fp64", 11)])
def test_whole_rounds(form, field):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    steps = 32
    L = B.rpdla_laser_init_intensity(0.8e-6, 2e-6, 4e-15, 1e21, t_before=0.5 * steps * DT,
                                     t_after=0.5 * steps * DT)
    L.field = field
    if field == 11:
        L.test_E[0], L.test_E[2], L.test_B[1] = 3e11, 1e12, 1e3
    prec = B.RPDLA_MIXED if form == "mixed" else B.RPDLA_FP64
    waves = int(B.rpdla_kernel_occupancy(B.RPDLA_KERNEL_PUSH, field, prec)["waves_per_simd"])
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    round_ = 64 * simds * waves
    for born in (2 * round_ - 64, 2 * round_, 2 * round_ + 65, 3 * round_ + round_ // 3):
        n = born + 1000
        rng = np.random.default_rng([born, field])
        z = rng.uniform(-10e-6, 10e-6, n)
        tb = z / 299792458.0 + 0.9 * steps * DT * rng.uniform(-0.5, 0.5, n)
        tb[rng.permutation(n)[:n - born]] = np.inf
        t, x, y, zz = (torch.as_tensor(a, device="cuda") for a in
                       (tb, rng.uniform(-3e-6, 3e-6, n), rng.uniform(-3e-6, 3e-6, n), z))
        print(f"{form} field {field}: {born} born slots, rounds of {round_}", flush=True)
        got = _push(B, form, L, t, (x, y, zz), 1)
        if form == "rr":
            _same(got, _other(torch, B, form, L, t, (x, y, zz), 1))
        else:
            _same(got, B.rpdla_push_noalloc(L, prec, t, x, y, zz, 1,
                                            tuple(torch.empty_like(t) for _ in range(6))))
        assert int(torch.isfinite(got[0]).sum()) == born


@pytest.mark.parametrize("precision,n", [(0, 40000), (1, 70000)])
def test_batched_whole_rounds(precision, n):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    n_cfg, kf, kl = 2, 1, 10
    lasers = [B.rpdla_laser_init_intensity(0.8e-6, 3e-6, 30e-15, I, t_before=30 * DT, t_after=30 * DT)
              for I in (1e21, 3e21)]
    arr = (B.rpdla_laser * n_cfg)(*lasers)
    spec = B.rpdla_hist_spec(32, 18, -6.0, 3.0, 0)
    full = B.rpdla_batched_workspace_bytes(n_cfg, n, kf, kl)
    lay = B.rpdla_batched_workspace_layout(n_cfg, n, kf, kl)
    chunk = lay["uz"] + (n_cfg * n * 10 * 8 + 255) // 256 * 256
    waves = int(B.rpdla_kernel_occupancy(B.RPDLA_KERNEL_BATCHED_PUSH, 5, precision)["waves_per_simd"])
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    got = []
    print(f"batched {n_cfg} x {n} atoms, precision {precision}", flush=True)
    for size in (full, chunk):
        counts = torch.zeros((n_cfg, 2, 32, 18), dtype=torch.int64, device="cuda")
        tallies = torch.zeros((n_cfg, 6), dtype=torch.int64, device="cuda")
        steps = torch.zeros(n_cfg, dtype=torch.int64, device="cuda")
        ws = torch.zeros(full, dtype=torch.uint8, device="cuda")
        st = B.lib.rpdla_run_batched(arr, n_cfg, 5, 40, n, n, 2.0, kf, kl, precision, C.byref(spec),
                                     counts.data_ptr(), tallies.data_ptr(), steps.data_ptr(),
                                     ws.data_ptr(), size, 0)
        assert st == B.RPDLA_OK, B.lib.rpdla_last_error()
        torch.cuda.synchronize()
        a = B.batched_chunk_arrays(ws, n_cfg, n, kf, kl)
        born = torch.isfinite(a["t_birth"])
        zero = torch.zeros((), dtype=torch.float64, device="cuda")
        got.append([counts, tallies, steps, a["t_birth"].clone()] +
                   [torch.where(born, a[k], zero) for k in ("ux", "uy", "uz")])
        assert int(born.sum()) > 2 * 64 * simds * waves
    for x, y in zip(*got):
        assert torch.equal(x.contiguous().view(torch.int64), y.contiguous().view(torch.int64))
