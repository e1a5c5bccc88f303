"""FP64 calls that evaluate each pair once for both partners (the default from
8192 particles on, and layout screen 2): as accurate as the ordered kernels,
whose separations they form in the same way.

Bar on |a_i - ref_i| / sum_j |a_ij|, in units of u = 2^-53: 16 for the
roundings of a pair's own term, and 32 for the sum of at most 1024 terms in
any order (a random walk of sqrt(1024) steps of u): 48 u = 5.3e-15.
"""
import numpy as np
import pytest

import oracle
from gpu_common import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu

BAR = 48 * 2.0 ** -53


@pytest.fixture(scope="module")
def env():
    torch, p3 = gpu_or_skip()
    ctx = p3.Context(0)
    ctx.set_tune_cache("")
    return torch, p3, ctx


# 3 tiles: every cluster meets images of the box; 18: most do not
@pytest.mark.parametrize("n,tiles", [(8192, 3), (32768, 18)])
@pytest.mark.parametrize("masses", [False, True])
@pytest.mark.parametrize("cfg", [{}, dict(cluster_size=16, screen=2), dict(cluster_size=32, screen=2),
                                 dict(cluster_size=64, screen=2)])
def test_separations_as_in_the_ordered_kernels(env, n, tiles, masses, cfg):
    torch, p3, ctx = env
    print("fp64 accuracy", n, tiles, masses, cfg, flush=True)
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3))
    # pairs across the box's faces, at coordinates of very different sizes
    pos[:400, 0] = np.where(np.arange(400) % 2, 1e-9 * rng.random(400), 1.0 - 1e-4 * rng.random(400))
    mass = rng.random(n) + 0.5 if masses else None
    r_cut = 1.0 / (tiles + 0.01)
    recv = np.concatenate([np.arange(400), np.arange(400, n, 17)])
    ref, cnt, absum, _ = oracle.force(pos, mass, 1.0, r_cut / 4.5, r_cut, recv=recv, method="tiled")
    m = int(cnt.max())
    ctx.set_config(**cfg)
    try:
        acc = ctx.force(to_dev(torch, pos), to_dev(torch, mass), None, box=1.0, x_s=r_cut / 4.5,
                        r_cut=r_cut, precision="fp64").cpu().numpy()
        assert ctx.stats()["screen"] == 2
    finally:
        ctx.set_config()
    e = oracle.errors(acc[recv], ref, absum)
    bar = max(BAR, (16 + np.sqrt(m)) * 2.0 ** -53)
    print(e, m, bar, flush=True)
    assert e["e_max_cond"] <= bar, (e, bar)
