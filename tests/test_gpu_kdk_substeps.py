"""KDK sub-steps with and without the host's wait for the due count: sets whose
top rung holds fewer particles than a wave, one that empties inside the period,
and one that stays full; sizes around the kernels' 1024-thread blocks.  Bars of
the other KDK tests."""
import numpy as np
import pytest

from gpu_common import gpu_or_skip
from test_gpu_kdk import eps_for, gpu_run, oracle_run, periodic_diff

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch, p3 = gpu_or_skip()
    return torch, p3, p3.Context(0)


def _compare(env, pos, vel, mass, dt, n_steps, eps, **kw):
    xo, vo, ro = oracle_run(pos, vel, mass, dt, n_steps, eps, **kw)
    xg, vg, rg, st = gpu_run(env, pos, vel, mass, dt, n_steps, eps, **kw)
    dv = np.max(np.abs(vo - vel))
    assert np.max(np.abs(periodic_diff(xg, xo))) <= 1e-11
    assert np.max(np.abs(vg - vo)) <= 1e-9 * dv
    assert np.array_equal(rg, ro)
    return st


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2500])
@pytest.mark.parametrize("clump", [8, 400])
def test_top_rung_small_and_large(env, n, clump):
    print("kdk top rung", n, clump, flush=True)
    rng = np.random.default_rng(n + clump)
    pos = rng.random((n, 3))
    pos[:clump] = (0.5 + 0.02 * (clump / 400) ** (1 / 3) * rng.standard_normal((clump, 3))) % 1.0
    vel = 0.05 * rng.standard_normal((n, 3))
    st = _compare(env, pos, vel, rng.uniform(0.5, 1.5, n) / n, 3e-3, 2, eps_for(n))
    assert st["sr_calls"] <= 1 + st["substeps"]


def test_top_rung_empties(env):
    """A fast pair flies apart: the rungs above the others empty inside the
    period, and the sub-steps without kicks are not counted as calls."""
    print("kdk emptying rung", flush=True)
    rng = np.random.default_rng(3)
    n = 500
    pos, vel = rng.random((n, 3)), np.zeros((n, 3))
    eps = eps_for(n)
    pos[0], pos[1] = [0.5, 0.5, 0.5], [0.5 + 2.0 * eps, 0.5, 0.5]
    vel[0, 0], vel[1, 0] = -30.0, 30.0
    mass = np.full(n, 1.0 / n)
    mass[:2] = 0.2
    st = _compare(env, pos, vel, mass, 3e-3, 2, eps)
    assert st["sr_calls"] < 1 + st["substeps"], st
