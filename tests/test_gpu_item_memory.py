"""Memory of the work items: it grows with the set and not with its square, and
a call whose dense tiles cannot be split for want of memory runs unsplit."""
import numpy as np
import pytest

from gpu_common import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return gpu_or_skip()


def _set(torch, n, seed=1):
    rng = np.random.default_rng(seed)
    pos = rng.random((n, 3))
    pos[: n // 50] = 0.5 + 0.01 * rng.random((n // 50, 3))
    act = (rng.random(n) < 0.3).astype(np.uint8)
    r_cut = 5.6 * 0.5 / n ** (1 / 3)
    return to_dev(torch, pos), to_dev(torch, act), dict(box=1.0, x_s=r_cut / 4.5, r_cut=r_cut)


def _call(ctx, pos, act, kw, kind, prec):
    return ctx.force(pos, None, act if kind == "mask" else None, precision=prec, **kw)


def _try(p3, det, limit, call):
    """The call's result on a new handle that may hold `limit` bytes, or None."""
    ctx = p3.Context(0)
    try:
        ctx.set_tune_cache("")
        ctx.set_deterministic(det)
        ctx.set_debug_limits(max_workspace_bytes=int(limit))
        try:
            return call(ctx), ctx.stats()
        except p3.P3MError as e:
            assert e.code == p3.P3M_ENOMEM, e
            return None
    finally:
        ctx.close()


@pytest.mark.parametrize("n", [30000, 250000])
@pytest.mark.parametrize("kind,prec", [("all", "fp64"), ("all", "fp32"), ("mask", "fp32")])
@pytest.mark.parametrize("det", [0, 1])
def test_small_limits(env, n, kind, prec, det):
    torch, p3 = env
    pos, act, kw = _set(torch, n)
    call = lambda ctx: _call(ctx, pos, act, kw, kind, prec)
    ref, st = _try(p3, det, 1 << 34, call)
    # the least memory the call runs with, to 2 %
    lo, hi = 1.0, 4000.0 * n
    while hi > 1.02 * lo:
        mid = (lo * hi) ** 0.5
        print("item memory", n, kind, prec, det, "limit", int(mid), flush=True)
        if _try(p3, det, mid, call) is None:
            lo = mid
        else:
            hi = mid
    got, st_low = _try(p3, det, hi, call)
    assert st_low["interactions"] == st["interactions"]
    assert float((got - ref).abs().max()) <= 1e-12 * float(ref.abs().max())
    # fixed parts about 160 bytes a particle (200 masked), unsplit items at
    # most 60 (120 masked, in clusters of 8); deterministic: the sort's 24,
    # and 24 bytes of partial sums per item and receiver (about two items)
    assert hi <= n * (400 if not det else 700), hi / n
    # and with the split at most 256 runs of a tile per cluster more
    csize = st["cluster_size"]
    if not det:
        assert _try(p3, det, hi + 1.3 * 256 * 16 * (n / csize + 30), call)[1]["items"] == st["items"]


def test_noalloc_deterministic_with_dense_tiles(env):
    """64 tiles of 1000 particles: split, their partial slots pass the fixed
    workspace; unsplit they fit."""
    torch, p3 = env
    print("no-alloc deterministic", flush=True)
    ctx = p3.Context(0)
    try:
        ctx.set_tune_cache("")
        n = 65000
        pos = to_dev(torch, np.random.default_rng(3).random((n, 3)))
        kw = dict(box=1.0, x_s=1.0 / 4.01 / 4.5, r_cut=1.0 / 4.01, precision="fp32")
        ref = ctx.force(pos, **kw)
        ctx.set_deterministic(1)
        got = ctx.force_noalloc(pos, **kw)
        assert float((got - ref).abs().max()) <= 1e-12 * float(ref.abs().max())
        assert torch.equal(got, ctx.force_noalloc(pos, **kw))
    finally:
        ctx.close()
