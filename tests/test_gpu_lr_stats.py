"""The long-range statistics after calls that failed to grow their workspace:
those of the last call that ran."""
import numpy as np
import pytest

from gpu_common import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("timing", [0, 1])
def test_stats_after_failed_growth(timing):
    torch, p3 = gpu_or_skip()
    rng = np.random.default_rng(2)
    small, large = to_dev(torch, rng.random((500, 3))), to_dev(torch, rng.random((40000, 3)))
    ref_ctx = p3.Context(0)
    ref = ref_ctx.force_long_range(large, box=1.0, n_grid=64, x_s=1.25 / 64)
    ref_ctx.close()
    failed = 0
    for k in range(20):
        print("long-range growth", k, flush=True)
        ctx = p3.Context(0)
        try:
            ctx.set_timing(timing)
            ctx.force_long_range(small, box=1.0, n_grid=16, x_s=1.25 / 16)
            first = ctx.lr_stats()
            assert first["n"] == 500 and first["n_grid"] == 16
            ctx.set_debug_limits(fail_after=k)
            try:
                ctx.force_long_range(large, box=1.0, n_grid=64, x_s=1.25 / 64)
                ok = True
            except p3.P3MError as e:
                assert e.code == p3.P3M_ENOMEM, e
                ok = False
                failed += 1
                assert ctx.lr_stats() == first
            ctx.set_debug_limits()
            got = ctx.force_long_range(large, box=1.0, n_grid=64, x_s=1.25 / 64)
            assert float((got - ref).abs().max()) <= 1e-12 * float(ref.abs().max())
            assert ctx.lr_stats()["n"] == 40000
        finally:
            ctx.close()
        if ok:
            break
    assert failed >= 5 and ok
