"""Dense tiles cut into runs of their records, in the smallest box (3 tiles per
dimension: the 27 tiles of a stencil are all of it): every run of every tile
met once, also of the own tile's upper part in the pairs-once layouts.  A run
lost or doubled changes the accepted-pair count."""
import numpy as np
import pytest

import oracle
from gpu_common import TOL, gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch, p3 = gpu_or_skip()
    ctx = p3.Context(0)
    ctx.set_tune_cache("")
    return torch, p3, ctx


# every tile above the item size, and half the particles in one tile
@pytest.mark.parametrize("shape", ["uniform", "clump"])
@pytest.mark.parametrize("tiles", [3, 4])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("csize,screen", [(16, 2), (32, 2), (64, 2), (8, 1), (32, 1), (64, 0)])
def test_runs(env, shape, tiles, prec, csize, screen):
    torch, p3, ctx = env
    print("split runs", shape, tiles, prec, csize, screen, flush=True)
    rng = np.random.default_rng(tiles)
    n = 3001
    pos, mass = rng.random((n, 3)), rng.random(n) + 0.5
    if shape == "clump":
        pos[: n // 2] = 0.01 + 0.2 * rng.random((n // 2, 3))
    act = (rng.random(n) < 0.3).astype(np.uint8)
    w = rng.standard_normal((n, 3))
    r_cut = 1.0 / (tiles + 0.01)
    kw = dict(box=1.0, x_s=r_cut / 4.5, r_cut=r_cut, precision=prec)
    d, m, a = to_dev(torch, pos), to_dev(torch, mass), to_dev(torch, act)
    ctx.set_config(subtiles_per_dim=1, item_target=64, cluster_size=csize, screen=screen)
    try:
        for sel, sel_np in ((None, None), (a, act)):
            got = ctx.force(d, m, sel, **kw).cpu().numpy()
            st = ctx.stats()
            ref, cnt, absum = oracle.force_full(pos, mass, 1.0, r_cut / 4.5, r_cut, active=sel_np)
            assert st["interactions"] == int(cnt.sum())
            assert st["items"] > st["clusters"]
            e = oracle.errors(got, ref, absum)
            assert e["e_l2"] <= TOL[prec] and e["e_max_cond"] <= TOL[prec], e
        g = ctx.force_backward(d, m, a, to_dev(torch, w), **kw).cpu().numpy()
        ref = oracle.vjp(pos, mass, act, w, 1.0, r_cut / 4.5, r_cut, method="tiled")
        assert np.linalg.norm(g - ref) <= TOL[prec] * np.linalg.norm(ref)
    finally:
        ctx.set_config()
