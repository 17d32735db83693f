"""The batched sweep's ordered push against its queue push, which a workspace
of the chunk's arrays alone still runs: bitwise the same births and momenta,
the same counts, tallies and steps, for part sizes around whole groups of 64,
partial last chunks, one and 64 configurations, few and no births, and more
groups than one wave per SIMD."""
import ctypes as C

import pytest

from gpu_common import require_gpu

pytestmark = pytest.mark.gpu

# configurations, atoms, atoms per chunk, first and last state, intensity [W/cm^2]
CASES = [(1, 1, 1, 8, 8, 1e21), (1, 64, 64, 1, 10, 1e21), (3, 13, 7, 1, 5, 1e21),
         (64, 9, 9, 1, 10, 1e21), (5, 129, 64, 7, 9, 3e19), (2, 50, 50, 9, 10, 1e18),
         (7, 1900, 1900, 1, 10, 1e21), (2, 14000, 14000, 1, 10, 1e21)]


@pytest.mark.parametrize("n_cfg,n,apc,kf,kl,I", CASES)
@pytest.mark.parametrize("precision", [0, 1])
def test_ordered_equals_queue(n_cfg, n, apc, kf, kl, I, precision):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    K = kl - kf + 1
    lasers = []
    for c in range(n_cfg):
        lam = (0.8 + 0.05 * (c % 9)) * 1e-6
        lasers.append(B.rpdla_laser_init_intensity(lam, 2.5 * lam, (2 + c % 3) * 1e-15,
                                                   I * (1 + c % 4)))
    arr = (B.rpdla_laser * n_cfg)(*lasers)
    spec = B.rpdla_hist_spec(32, 18, -4.0, 3.0, 0)
    full = B.rpdla_batched_workspace_bytes(n_cfg, apc, kf, kl)
    lay = B.rpdla_batched_workspace_layout(n_cfg, apc, kf, kl)
    chunk = lay["uz"] + (n_cfg * apc * K * 8 + 255) // 256 * 256
    assert chunk < full
    stream = torch.cuda.Stream()
    got = []
    print(f"batched {n_cfg} x {n} atoms, chunks of {apc}, precision {precision}", flush=True)
    for size in (full, chunk):
        counts = torch.zeros((n_cfg, 2, 32, 18), dtype=torch.int64, device="cuda")
        tallies = torch.zeros((n_cfg, 6), dtype=torch.int64, device="cuda")
        steps = torch.zeros(n_cfg, dtype=torch.int64, device="cuda")
        ws = torch.zeros(full, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        for _ in range(2):                   # a graph capture, then a replay
            st = B.lib.rpdla_run_batched(
                arr, n_cfg, 5, 40, n, apc, 2.0, kf, kl, precision, C.byref(spec),
                C.c_void_p(counts.data_ptr()), C.c_void_p(tallies.data_ptr()),
                C.c_void_p(steps.data_ptr()), C.c_void_p(ws.data_ptr()), C.c_size_t(size),
                C.c_void_p(stream.cuda_stream))
            assert st == B.RPDLA_OK, B.lib.rpdla_last_error()
        stream.synchronize()
        last = n - (n - 1) // apc * apc      # atoms of the last chunk
        a = B.batched_chunk_arrays(ws, n_cfg, apc, kf, kl)
        tb = a["t_birth"][:, :last].clone()
        born = torch.isfinite(tb)
        zero = torch.zeros((), dtype=torch.float64, device="cuda")
        got.append([counts, tallies, steps, tb] +
                   [torch.where(born, a[k][:, :last], zero) for k in ("ux", "uy", "uz")])
    for x, y in zip(*got):
        assert torch.equal(x.contiguous().view(torch.int64), y.contiguous().view(torch.int64))
    # forward, backward, unborn and NaN: every slot once a run
    assert int(got[0][1][:, [0, 1, 4, 5]].sum()) == 2 * n_cfg * n * K
