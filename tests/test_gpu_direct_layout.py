"""Layouts that a configuration sets in part: calls configured to walk their
suppliers directly (screen 0) take the clusters the direct walk is fast with,
and every partly set layout gives the same sums."""
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


# 2^17: clusters of 64; with fewer than three subtiles per dimension the FP64
# adjoint from 3 * 2^18 on, masked receivers not at all
@pytest.mark.parametrize("n", [5000, (1 << 17) - 1, 1 << 17, 3 << 18])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("cfg", [dict(screen=0), dict(screen=0, subtiles_per_dim=2),
                                 dict(screen=0, subtiles_per_dim=3), dict(screen=0, item_target=512),
                                 dict(subtiles_per_dim=2), dict(item_target=512),
                                 dict(cluster_size=64), dict(screen=0, cluster_size=16)])
def test_partly_set_layouts(env, n, prec, cfg):
    torch, p3, ctx = env
    print("partly set", n, prec, cfg, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    pos = torch.rand((n, 3), generator=gen, device="cuda", dtype=torch.float64)
    w = torch.randn((n, 3), generator=gen, device="cuda", dtype=torch.float64)
    mask = (torch.rand(n, generator=gen, device="cuda") < 0.3).to(torch.uint8)
    rung = torch.randint(0, 3, (n,), generator=gen, device="cuda").to(torch.uint8)
    r_cut = 2.0 / n ** (1 / 3)
    kw = dict(box=1.0, x_s=r_cut / 4.5, r_cut=r_cut, precision=prec)
    calls = {"all": lambda: ctx.force(pos, None, None, **kw),
             "mask": lambda: ctx.force(pos, None, mask, **kw),
             "batched": lambda: ctx.force_batched(pos, None, rung, [0, 1, 2], **kw),
             "adjoint": lambda: ctx.force_backward(pos, None, None, w, **kw)}
    for name, call in calls.items():
        # the same arithmetic: the FP32 adjoint's differs between direct and screened walks
        full = dict(subtiles_per_dim=1, item_target=1024, cluster_size=32, screen=0)
        ctx.set_config(**full)
        try:
            ref, st_ref = call(), ctx.stats()
            ctx.set_config(**cfg)
            got, st = call(), ctx.stats()
        finally:
            ctx.set_config()
        assert st["interactions"] == st_ref["interactions"], name
        bar = 1e-12 if prec == "fp64" or name != "adjoint" or st["screen"] == 0 else 1e-5
        assert float((got - ref).abs().max()) <= bar * float(ref.abs().max()), name
        if cfg.get("screen") == 0:
            assert st["screen"] == 0
            if "cluster_size" not in cfg:
                fp32_adjoint = name == "adjoint" and prec == "fp32"
                fine = cfg.get("subtiles_per_dim", 1) >= 3
                from_n = (3 << 18) if name == "adjoint" and not fine else (1 << 17)
                wide = n >= from_n and (name != "mask" or fine)
                assert (st["cluster_size"] == 64) == (wide or fp32_adjoint), (name, st)
