"""The long-range deposit and readout at the edges of their bins: bins of
exactly 2048 particles and around it (longer ones are finished run by run), a
set in a single bin, and particles on the bins' and the box's borders."""
import numpy as np
import pytest

from gpu_common import gpu_or_skip, to_dev
from oracle import pm_oracle as pm

pytestmark = pytest.mark.gpu

# FP64 throughout: the bar of the other long-range tests
TOL_PM = 1e-12


@pytest.fixture(scope="module")
def env():
    torch, p3 = gpu_or_skip()
    return torch, p3, p3.Context(0)


def _check(env, pos, mass, n_grid, active=None):
    torch, p3, ctx = env
    x_s = 1.25 / n_grid
    got = ctx.force_long_range(to_dev(torch, pos), to_dev(torch, mass), to_dev(torch, active),
                               box=1.0, n_grid=n_grid, x_s=x_s).cpu().numpy()
    ref = pm.pm_force(pos, mass, 1.0, n_grid, x_s, active=active)
    assert np.max(np.abs(got - ref)) <= TOL_PM * np.max(np.abs(ref))
    ctx.lr_stats()   # raises if the bin scan gave up


@pytest.mark.parametrize("n_grid", [16, 32, 64])
@pytest.mark.parametrize("dense", [2047, 2048, 2049, 4096, 6200])
@pytest.mark.parametrize("corner", [0.0, 0.5])
def test_dense_bin(env, n_grid, dense, corner):
    """`dense` particles around one bin's corner, at the box border and inside."""
    print("dense bin", n_grid, dense, corner, flush=True)
    rng = np.random.default_rng(dense + n_grid)
    side = 8.0 / n_grid
    clump = corner + side * (0.0 if corner == 0.0 else -0.25) + 0.9 * side * rng.random((dense, 3))
    pos = np.concatenate([clump, rng.random((300, 3))]) % 1.0
    active = (rng.random(len(pos)) < 0.8).astype(np.uint8)
    _check(env, pos, rng.random(len(pos)) + 0.5, n_grid, active)


@pytest.mark.parametrize("n_grid", [16, 32, 128])
def test_borders(env, n_grid):
    """Particles on nodes, half way between them, and on both ends of the box."""
    print("borders", n_grid, flush=True)
    h = 1.0 / n_grid
    q = np.array([0.0, 0.25 * h, 0.5 * h, h, 7.5 * h, 8.0 * h, 8.5 * h, 15.5 * h, 0.5, 1.0 - h,
                  1.0 - 0.5 * h, 1.0 - 1e-16])
    pos = np.stack(np.meshgrid(q, q, q, indexing="ij"), -1).reshape(-1, 3)
    _check(env, pos, 1.0 + np.arange(len(pos)) % 7 / 7.0, n_grid)
