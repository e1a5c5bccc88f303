"""KDK steps whose top rung starts with more than a wave of particles, all of
which leave it inside the period: the sub-steps without kicks are queued as
force calls without receivers, and in sets above 2^17 particles asked about
from the first one on.  Bars of the other KDK tests."""
import numpy as np
import pytest

import oracle
from gpu_common import gpu_or_skip, to_dev
from oracle import kdk_oracle as kdk

pytestmark = pytest.mark.gpu

R_CUT = 1.0 / 40.01
X_S = R_CUT / 4.5
EPS, DT = 1e-4, 1e-3


@pytest.mark.parametrize("n,n_steps", [(3000, 1), (3000, 2), ((1 << 17) - 1, 1), (1 << 17, 1),
                                       ((1 << 17) + 1, 1), (140000, 1), (140000, 2)])
def test_top_rung_empties(n, n_steps):
    torch, p3 = gpu_or_skip()
    print("kdk emptying", n, n_steps, flush=True)
    rng = np.random.default_rng(n)
    pos, vel = rng.random((n, 3)), np.zeros((n, 3))
    mass = np.full(n, 1e-12)
    # 125 pairs that fly apart by 10 eps in the first sub-step of dt / 16
    site = (np.stack(np.meshgrid(*3 * [np.arange(5)], indexing="ij"), -1).reshape(-1, 3) + 0.5) / 5
    pos[0:250:2], pos[1:250:2] = site, site + [2 * EPS, 0, 0]
    vel[0:250:2, 0], vel[1:250:2, 0] = -80 * EPS / DT, 80 * EPS / DT
    mass[:250] = 2.84e-5

    def sr(x, active):
        return oracle.force_full(x, mass, 1.0, X_S, R_CUT, active=active, eps=EPS)[0]

    xo, vo, ro = kdk.kdk(pos, vel, 1.0, DT, n_steps, sr, eps=EPS)
    ctx = p3.Context(0)
    try:
        p, v, r = to_dev(torch, pos), to_dev(torch, vel), to_dev(torch, np.zeros(n, np.uint8))
        ctx.kdk_step(p, v, to_dev(torch, mass), r, box=1.0, x_s=X_S, r_cut=R_CUT, n_grid=0, dt=DT,
                     n_steps=n_steps, eps=EPS)
        st, sr_st = ctx.kdk_stats(), ctx.stats()
    finally:
        ctx.close()
    assert st["highest_rung"] >= 3 and st["sr_calls"] < 1 + st["substeps"], st
    assert sr_st["receivers"] == n   # of the last sub-step, which kicks everyone
    d = p.cpu().numpy() - xo
    assert np.max(np.abs(d - np.round(d))) <= 1e-11
    assert np.max(np.abs(v.cpu().numpy() - vo)) <= 1e-9 * np.max(np.abs(vo - vel))
    assert np.array_equal(r.cpu().numpy(), ro)
