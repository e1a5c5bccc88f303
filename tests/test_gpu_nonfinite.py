"""Infinite and NaN masses and gradients, FP64: they reach the particles within
r_cut of their own and no others, whichever layout a call takes."""
import numpy as np
import pytest

import oracle
from gpu_common import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch, p3 = gpu_or_skip()
    ctx = p3.Context(0)
    ctx.set_tune_cache("")
    return torch, p3, ctx


# 8192: each pair once for both partners by default, below it the ordered kernels
@pytest.mark.parametrize("n", [4000, 8192])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("cfg", [{}, dict(cluster_size=32, screen=2), dict(cluster_size=16, screen=1)])
@pytest.mark.parametrize("eps", [0.0, 0.002])
def test_reach(env, n, value, cfg, eps):
    torch, p3, ctx = env
    print("nonfinite", n, value, cfg, eps, flush=True)
    rng = np.random.default_rng(n)
    pos, mass, w = rng.random((n, 3)), rng.random(n) + 0.5, rng.standard_normal((n, 3))
    bad = np.array([5, n // 2, n - 1])
    r_cut = 1.0 / 9.01
    d = pos[:, None, :] - pos[None, bad, :]
    d -= np.round(d)
    r2 = oracle.sq_dist(d.reshape(-1, 3)).reshape(n, -1)
    near = ((r2 < r_cut * r_cut) & (r2 > 0)).any(1)
    kw = dict(box=1.0, x_s=r_cut / 4.5, r_cut=r_cut, precision="fp64")
    mass_bad, w_bad = mass.copy(), w.copy()
    mass_bad[bad] = value
    w_bad[bad] = value
    ctx.set_config(**cfg)
    ctx.set_softening(eps)
    try:
        a = ctx.force(to_dev(torch, pos), to_dev(torch, mass_bad), None, **kw).cpu().numpy()
        g = ctx.force_backward(to_dev(torch, pos), to_dev(torch, mass), None, to_dev(torch, w_bad),
                               **kw).cpu().numpy()
        # rows beyond the reach are those of a call without the values
        ok = ctx.force(to_dev(torch, pos), to_dev(torch, mass), None, **kw).cpu().numpy()
    finally:
        ctx.set_config()
        ctx.set_softening(0.0)
    assert np.array_equal(~np.isfinite(a).all(1), near)
    assert np.max(np.abs(a - ok)[~near]) <= 1e-12 * np.max(np.abs(ok))
    own = np.zeros(n, bool)
    own[bad] = True
    assert np.array_equal(~np.isfinite(g).all(1), near | own)
