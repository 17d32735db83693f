"""The kernels that rpdla_push and rpdla_run_batched run keep every value in
registers, at every field order, and reach the waves they are compiled for."""
import pytest

from gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field", [1, 3, 5, 10, 11, 21, 23, 25])
def test_no_scratch(field):
    require_gpu()
    from paper_2509_01741_amd import binding as B
    fp64 = 3 if field in (23, 25) else 4
    for kind in (B.RPDLA_KERNEL_PUSH, B.RPDLA_KERNEL_BATCHED_PUSH):
        for prec, waves in ((B.RPDLA_FP64, fp64), (B.RPDLA_MIXED, 7)):
            if field > 20 and prec == B.RPDLA_MIXED:
                continue
            r = B.rpdla_kernel_occupancy(kind, field, prec)
            print(f"field {field} kind {kind} precision {prec}: {r}", flush=True)
            assert r["scratch_bytes"] == 0 and r["waves_per_simd"] >= waves
            assert 0 < r["vgprs"] <= 512 // waves
