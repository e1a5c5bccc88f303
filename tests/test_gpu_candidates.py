"""The candidates counter of FP64 calls: (receiver, supplier) pairs handed to
the pair loop, which hold every accepted pair, in each layout."""
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


@pytest.mark.parametrize("n", [4000, 8192, 30000])
@pytest.mark.parametrize("cfg", [{}, dict(cluster_size=16, screen=2), dict(cluster_size=64, screen=2)])
@pytest.mark.parametrize("backward", [False, True])
def test_candidates_hold_the_accepted_pairs(env, n, cfg, backward):
    torch, p3, ctx = env
    print("candidates", n, cfg, backward, flush=True)
    rng = np.random.default_rng(n)
    pos = to_dev(torch, rng.random((n, 3)))
    w = to_dev(torch, rng.standard_normal((n, 3)))
    r_cut = 1.0 / 11.01
    kw = dict(box=1.0, x_s=r_cut / 4.5, r_cut=r_cut, precision="fp64")
    ctx.set_config(**cfg)
    try:
        if backward:
            ctx.force_backward(pos, None, None, w, **kw)
        else:
            ctx.force(pos, None, None, **kw)
        st = ctx.stats()
    finally:
        ctx.set_config()
    # at most every particle of the 27 tiles around each one
    assert st["interactions"] <= st["candidates"] <= 3 * 27 * n * (n / 11 ** 3)
