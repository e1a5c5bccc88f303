"""Receiver compaction and work planning at the edges of their blocks: the
tile counts where the plan changes its block (2^14 tiles), tiles holding more
clusters than a block plans at once or keeps counts of, and receiver rows
around the compaction's 16384-row tiles.  A cluster or an item lost, doubled
or misplaced changes the accepted-pair count or a receiver's force."""
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


def _check(env, pos, active, r_cut, prec, cfg, mass=None):
    torch, p3, ctx = env
    x_s = r_cut / 4.5
    ctx.set_config(**cfg)
    try:
        acc = ctx.force(to_dev(torch, pos), to_dev(torch, mass), to_dev(torch, active), box=1.0,
                        x_s=x_s, r_cut=r_cut, precision=prec).cpu().numpy()
        st = ctx.stats()
    finally:
        ctx.set_config()
    ref, cnt, absum = oracle.force_full(pos, mass, 1.0, x_s, r_cut, active=active)
    assert st["interactions"] == int(cnt.sum())
    assert st["receivers"] == (len(pos) if active is None else int(active.sum()))
    e = oracle.errors(acc, ref, absum)
    assert e["e_l2"] <= TOL[prec] and e["e_max_cond"] <= TOL[prec], e
    if active is not None:
        assert np.all(acc[active == 0] == 0)


# 64 and 125 tiles; 4096 and 4913 (the key kernel scans up to 4096 cells); 15625 and 17576
@pytest.mark.parametrize("nt", [4, 5, 16, 17, 25, 26])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("cfg", [dict(subtiles_per_dim=1, item_target=64, cluster_size=8, screen=1),
                                 dict(subtiles_per_dim=2, item_target=128, cluster_size=16, screen=2)])
def test_tile_counts(env, nt, masked, cfg):
    print("tiles", nt, masked, cfg, flush=True)
    rng = np.random.default_rng(nt)
    pos = rng.random((4000, 3))
    active = (rng.random(4000) < 0.3).astype(np.uint8) if masked else None
    _check(env, pos, active, 1.0 / (nt + 0.01), "fp64", cfg, mass=rng.random(4000) + 0.5)


@pytest.mark.parametrize("cfg", [dict(subtiles_per_dim=1, item_target=4096, cluster_size=8, screen=1),
                                 dict(subtiles_per_dim=3, item_target=64, cluster_size=8, screen=0),
                                 dict(subtiles_per_dim=1, item_target=1024, cluster_size=16, screen=2)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_dense_tile(env, cfg, prec):
    """9000 particles of one tile: 1125 clusters of 8."""
    print("dense tile", cfg, prec, flush=True)
    rng = np.random.default_rng(7)
    pos = np.concatenate([0.41 + 0.17 * rng.random((9000, 3)), rng.random((500, 3))])
    _check(env, pos, None, 1.0 / 5.01, prec, cfg)


@pytest.mark.parametrize("n", [16383, 16384, 16385, 40000])
def test_receiver_rows(env, n):
    """Batched rows 3 n around multiples of 16384 against single masked calls."""
    torch, p3, ctx = env
    print("receiver rows", n, flush=True)
    rng = np.random.default_rng(n)
    pos, rung = rng.random((n, 3)), rng.integers(0, 4, n).astype(np.uint8)
    r_cut = 1.0 / 12.01
    kw = dict(box=1.0, x_s=r_cut / 4.5, r_cut=r_cut, precision="fp64")
    thr = [1, 0, 3]
    out = ctx.force_batched(to_dev(torch, pos), None, to_dev(torch, rung), thr, **kw).cpu().numpy()
    st = ctx.stats()
    assert st["receivers"] == sum(int((rung >= k).sum()) for k in thr)
    ref, cnt, absum = oracle.force_full(pos, None, 1.0, r_cut / 4.5, r_cut)
    assert st["interactions"] == sum(int(cnt[rung >= k].sum()) for k in thr)
    for k, t in enumerate(thr):
        on = rung >= t
        e = oracle.errors(out[k][on], ref[on], absum[on])
        assert e["e_l2"] <= TOL["fp64"] and e["e_max_cond"] <= TOL["fp64"], (t, e)
        assert np.all(out[k][~on] == 0)
