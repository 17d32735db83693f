"""Launch shapes belong to the queue forms of the push: the autotuner times
those (its figures are those of rpdla_push_noalloc, not of the ordered
rpdla_push), stores the fastest of its figures, and every shape gives the same
bits in each call that runs a queue; the ordered push is not slower for a shape
that some queue asked for."""
import time

import numpy as np
import pytest

import seeded_inputs as SI
from gpu_common import require_gpu

pytestmark = pytest.mark.gpu


def _slots(torch, B, n, K):
    L = B.rpdla_laser_init_intensity(0.8e-6, 2e-6, 4e-15, 1e21)
    xs, ys, zs = SI.cylinder_atoms(n, n, 4e-6, 10e-6)
    rng = np.random.default_rng(n)
    tb = (zs[:, None] / 299792458.0 + 1e-15 * rng.normal(size=(n, K))).ravel()
    return L, [torch.as_tensor(a, device="cuda") for a in (tb, xs, ys, zs)]


def _ms(torch, f):
    f()
    best = 1e9
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, 1e3 * (time.perf_counter() - t))
    return best


def test_autotune_times_the_queue():
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    n, K = 2048, 10
    L = B.rpdla_laser_init_intensity(0.8e-6, 3e-6, 10e-15, 1e21)
    keep = [B.rpdla_get_launch_shape(k, 5, 0) for k in range(3)]
    try:
        rep = B.rpdla_autotune(L, 0, n, 1, K)
        for kind, key in ((B.RPDLA_KERNEL_PUSH, "push"), (B.RPDLA_KERNEL_BATCHED_PUSH, "batched_push")):
            best = min(rep[key + "_ms"], key=rep[key + "_ms"].get)
            assert rep[key + "_best"] == best
            assert "%dx%d" % B.rpdla_get_launch_shape(kind, 5, 0) == best
    finally:
        for k, s in enumerate(keep):
            B.rpdla_set_launch_shape(k, 5, 0, *s)
    # the probe's own slots, through both forms
    x, y, z = B.rpdla_sample_atoms(0x5eed, 0xA070, 0, n, 2 * L.w0, B.rpdla_rayleigh(L))
    tb = B.rpdla_ionize(L, 0x5eed, 0xA070, 0, x, y, z, 1, K)
    out = tuple(torch.empty_like(tb) for _ in range(6))
    queue = _ms(torch, lambda: B.rpdla_push_noalloc(L, 0, tb, x, y, z, K, out))
    ordered = _ms(torch, lambda: B.rpdla_push(L, 0, tb, x, y, z, K, out))
    got = rep["push_ms"]["256x1"]
    print(f"queue {queue:.2f} ms, ordered {ordered:.2f} ms, autotune 256x1 {got:.2f} ms", flush=True)
    assert abs(np.log(got / queue)) < abs(np.log(got / ordered))


@pytest.mark.parametrize("prec", [0, 1])
def test_shapes_give_the_same_bits(prec):
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    n, K = 301, 3
    L, (tb, *xyz) = _slots(torch, B, n, K)
    A = B.adaptive_settings()
    lay = B.rpdla_batched_workspace_layout(1, 40, 1, 10)
    chunk = lay["uz"] + (40 * 10 * 8 + 255) // 256 * 256
    got = []
    try:
        for blk, gf in ((64, 1), (256, 2), (128, 1), (192, 8)):
            for p in (0, prec):
                B.rpdla_set_launch_shape(B.RPDLA_KERNEL_PUSH, 5, p, blk, gf)
            B.rpdla_set_launch_shape(B.RPDLA_KERNEL_BATCHED_PUSH, 5, prec, blk, gf)
            out = tuple(torch.full_like(tb, 7.0) for _ in range(6))
            o = list(B.rpdla_push_noalloc(L, prec, tb, *xyz, K, out))
            o += list(B.rpdla_push_adaptive(L, A, tb, *xyz, K))
            ws = torch.zeros(chunk, dtype=torch.uint8, device="cuda")
            o += list(B.rpdla_run_batched([L], 5, 1, 40, 40, 2.0, 1, 10, prec,
                                          B.rpdla_hist_spec(32, 18, -3.0, 4.0, 0), workspace=ws))
            got.append([v.cpu().numpy() for v in o])
    finally:
        for p in (0, prec):
            B.rpdla_set_launch_shape(B.RPDLA_KERNEL_PUSH, 5, p, 256, 1)
        B.rpdla_set_launch_shape(B.RPDLA_KERNEL_BATCHED_PUSH, 5, prec, 256, 1)
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")


def test_ordered_push_ignores_the_shape():
    torch = require_gpu()
    from paper_2509_01741_amd import binding as B
    n = 100_000
    L, (tb, *xyz) = _slots(torch, B, n, 1)
    out = tuple(torch.empty_like(tb) for _ in range(6))
    push = lambda: B.rpdla_push(L, 0, tb, *xyz, 1, out)        # noqa: E731
    plain = _ms(torch, push)
    try:
        B.rpdla_set_launch_shape(B.RPDLA_KERNEL_PUSH, 5, 0, 128, 1)
        other = _ms(torch, push)
    finally:
        B.rpdla_set_launch_shape(B.RPDLA_KERNEL_PUSH, 5, 0, 256, 1)
    print(f"1e5 slots: {plain:.2f} ms, with the queue's block at 128 {other:.2f} ms", flush=True)
    assert other < 1.3 * plain
