"""Calls that neither a configuration nor the tuner decides, at the sizes where
their layout rule changes, against the unscreened layout of 64-receiver
clusters: the same accepted pairs and, FP32 pair terms being rounded alike on
both, the same sums to FP64 rounding."""
import numpy as np
import pytest

from gpu_common import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch, p3 = gpu_or_skip()
    ctx = p3.Context(0)
    ctx.set_tune_cache("")
    return torch, p3, ctx


def _points(n, shape, rng):
    if shape == "uniform":
        return rng.random((n, 3))
    # a quarter of the particles in one tile, which the plan splits by records
    m = n // 4
    return np.concatenate([0.45 + 0.04 * rng.random((m, 3)), rng.random((n - m, 3))])


# 2^14 and 2^16: item sizes; 8192: pairs once for both partners (FP64), wider
# clusters (FP32)
@pytest.mark.parametrize("n", [1, 700, 8191, 8192, 16383, 16384, 65535, 65537])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", ["uniform", "clump"])
def test_default_equals_direct_layout(env, n, prec, shape):
    torch, p3, ctx = env
    print("default layout", n, prec, shape, flush=True)
    rng = np.random.default_rng(n)
    pos = to_dev(torch, _points(n, shape, rng))
    mass = to_dev(torch, rng.random(n) + 0.5)
    mask = to_dev(torch, (rng.random(n) < 0.2).astype(np.uint8))
    rung = to_dev(torch, rng.integers(0, 4, n).astype(np.uint8))
    w = to_dev(torch, rng.standard_normal((n, 3)))
    r_cut = 1.0 / 17.01
    kw = dict(box=1.0, x_s=r_cut / 4.5, r_cut=r_cut, precision=prec)
    calls = {
        "all": lambda: ctx.force(pos, mass, None, **kw),
        "unit": lambda: ctx.force(pos, None, None, **kw),
        "mask": lambda: ctx.force(pos, mass, mask, **kw),
        "noalloc": lambda: ctx.force_noalloc(pos, mass, None, **kw),
        "batched": lambda: ctx.force_batched(pos, mass, rung, [0, 2, 3], **kw),
        "adjoint": lambda: ctx.force_backward(pos, mass, None, w, **kw),
        "adjoint mask": lambda: ctx.force_backward(pos, mass, mask, w, **kw),
    }
    for eps in (0.0, 0.002):
        for det in (0, 1):
            ctx.set_softening(eps)
            ctx.set_deterministic(det)
            try:
                for name, call in calls.items():
                    got, st = call(), ctx.stats()
                    ctx.set_config(subtiles_per_dim=2, item_target=1024, cluster_size=64, screen=0)
                    ref, st_ref = call(), ctx.stats()
                    ctx.set_config()
                    assert st["interactions"] == st_ref["interactions"], (name, eps, det)
                    assert st["receivers"] == st_ref["receivers"], (name, eps, det)
                    scale = float(ref.abs().max())
                    diff = float((got - ref).abs().max())
                    # FP64 sums in another order, and the rounding of the
                    # separations the mutual kernel forms from offsets
                    assert diff <= 1e-12 * scale, (name, eps, det, diff, scale)
            finally:
                ctx.set_config()
                ctx.set_softening(0.0)
                ctx.set_deterministic(0)


@pytest.mark.parametrize("n", [1 << 17, (1 << 17) + 1, 1 << 18])
@pytest.mark.parametrize("tiles", [3, 20, 50])
def test_noalloc_limits(env, n, tiles):
    """The fixed workspace still holds its largest calls, all active and masked."""
    torch, p3, ctx = env
    print("noalloc", n, tiles, flush=True)
    if tiles == 3 and n > 1 << 17:
        r_cut = 1.0 / 6.01   # 3 tiles hold 1e10 pairs at this size
    else:
        r_cut = 1.0 / (tiles + 0.01) if tiles > 3 else 1.0 / 4.01
    gen = torch.Generator(device="cuda").manual_seed(5)
    pos = torch.rand((n, 3), generator=gen, device="cuda", dtype=torch.float64)
    mask = (torch.rand(n, generator=gen, device="cuda") < 0.5).to(torch.uint8)
    for prec in ("fp32", "fp64"):
        for act in (None, mask):
            kw = dict(box=1.0, x_s=r_cut / 4.5, r_cut=r_cut, precision=prec)
            out = ctx.force_noalloc(pos, None, act, **kw)
            ref = ctx.force(pos, None, act, **kw)
            assert float((out - ref).abs().max()) <= 1e-12 * float(ref.abs().max())
