"""A sweep through the binding with a workspace of the chunk's arrays alone,
which the library takes (its push then runs from work counters): the same
births, counts, tallies and steps as with a full one, also through
pipeline.run_sweep; a workspace one byte smaller is refused."""
import pytest

from gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_cfg,apc,kf,kl", [(1, 1, 8, 8), (3, 20, 1, 10)])
def test_workspace_of_the_chunk(n_cfg, apc, kf, kl):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    from paper_2509_01741_amd import pipeline as P
    from paper_2509_01741_amd import workloads as W
    lay = B.rpdla_batched_workspace_layout(n_cfg, apc, kf, kl)
    chunk = lay["uz"] + (n_cfg * apc * (kl - kf + 1) * 8 + 255) // 256 * 256
    assert chunk < B.rpdla_batched_workspace_bytes(n_cfg, apc, kf, kl)
    wl = dict(W.SWEEP_FP64, lasers=[dict(lam=0.8e-6, w0=2e-6, tau=(2 + c) * 1e-15, P=1e15)
                                    for c in range(n_cfg)],
              atoms=apc, chunk=apc, k_first=kf, k_last=kl, field_order=5, seed=3)
    got = []
    for ws in (None, torch.empty(chunk, dtype=torch.uint8, device="cuda")):
        steps = torch.zeros(n_cfg, dtype=torch.int64, device="cuda")
        c, t = P.run_sweep(wl, B.RPDLA_FP64, workspace=ws, electron_steps=steps)[:2]
        got.append((c, t, steps))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    assert int(got[0][2].sum()) > 0
    with pytest.raises(ValueError):
        P.run_sweep(wl, B.RPDLA_FP64,
                    workspace=torch.empty(chunk - 1, dtype=torch.uint8, device="cuda"))
