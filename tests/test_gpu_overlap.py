"""Outputs that share memory with an input of the same call: the inputs are read
before the output is written, so the result is that of separate buffers."""
import ctypes

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


R_CUT = 1.0 / 12.01
N_GRID = 32


def _kw(prec):
    return dict(box=1.0, x_s=R_CUT / 4.5, r_cut=R_CUT, precision=prec)


def _close(got, ref):
    # the same call on other buffers: FP64 sums in another order
    assert float((got - ref).abs().max()) <= 1e-12 * float(ref.abs().max())


# 8192: the FP64 default evaluates each pair once for both partners
@pytest.mark.parametrize("n", [700, 9001])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("det", [0, 1])
def test_forward_over_inputs(env, n, prec, det):
    torch, p3, ctx = env
    print("overlap forward", n, prec, det, flush=True)
    rng = np.random.default_rng(n)
    pos, mass = to_dev(torch, rng.random((n, 3))), to_dev(torch, rng.random(n) + 0.5)
    act = to_dev(torch, (rng.random(n) < 0.4).astype(np.uint8))
    kw = _kw(prec)
    ctx.set_deterministic(det)
    try:
        for call in (ctx.force, ctx.force_noalloc):
            for sel in (None, act):
                ref = call(pos, mass, sel, **kw)
                over = pos.clone()
                _close(call(over, mass, sel, out=over, **kw), ref)
                # masses and mask inside the output's memory, at its end
                out = torch.empty((n, 3), dtype=torch.float64, device=pos.device)
                m = out.view(-1)[2 * n:]
                m.copy_(mass)
                _close(call(pos, m, sel, out=out, **kw), ref)
                if sel is not None:
                    s = out.view(torch.uint8).view(-1)[8 * n:9 * n]
                    s.copy_(sel)
                    _close(call(pos, mass, s, out=out, **kw), ref)
        rung = to_dev(torch, rng.integers(0, 3, n).astype(np.uint8))
        ref = ctx.force_batched(pos, mass, rung, [0, 1, 2], **kw)
        big = torch.empty((3, n, 3), dtype=torch.float64, device=pos.device)
        big[1].copy_(pos)
        _close(ctx.force_batched(big[1], mass, rung, [0, 1, 2], out=big, **kw), ref)
    finally:
        ctx.set_deterministic(0)


@pytest.mark.parametrize("n", [700, 9001])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_backward_over_inputs(env, n, prec):
    torch, p3, ctx = env
    print("overlap backward", n, prec, flush=True)
    rng = np.random.default_rng(n)
    pos, w = to_dev(torch, rng.random((n, 3))), to_dev(torch, rng.standard_normal((n, 3)))
    kw = _kw(prec)
    ref = ctx.force_backward(pos, None, None, w, **kw)
    lib = p3.load_library()

    def raw(p, g, out):
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        rc = lib.p3m_sr_force_backward(ctx._h, p.data_ptr(), None, None, n, 1.0, R_CUT / 4.5, R_CUT,
                                       p3.P3M_FP64 if prec == "fp64" else p3.P3M_FP32,
                                       g.data_ptr(), out.data_ptr(), stream)
        assert rc == 0
        return out

    over = w.clone()
    _close(raw(pos, over, over), ref)
    over = pos.clone()
    _close(raw(over, w, over), ref)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_long_range_and_whole_force_over_positions(env, prec):
    torch, p3, ctx = env
    print("overlap whole force", prec, flush=True)
    n = 20000
    rng = np.random.default_rng(4)
    pos = to_dev(torch, rng.random((n, 3)))
    ref = ctx.force_long_range(pos, box=1.0, n_grid=N_GRID, x_s=R_CUT / 4.5)
    over = pos.clone()
    _close(ctx.force_long_range(over, box=1.0, n_grid=N_GRID, x_s=R_CUT / 4.5, out=over), ref)
    ref = ctx.force_total(pos, n_grid=N_GRID, **_kw(prec))
    for _ in range(5):
        over = pos.clone()
        _close(ctx.force_total(over, n_grid=N_GRID, out=over, **_kw(prec)), ref)
