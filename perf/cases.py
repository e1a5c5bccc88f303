"""Work that programs have this library do, as cases a timing harness can run.

Every case is one call (or one forward and backward pair) through the public
entry points, on synthetic particle sets shaped like the ones the P3M set-up
is used with: a unit periodic box, a mesh spacing of half the mean particle
distance, x_s = 1.25 mesh cells and r_cut = 4.5 x_s, and particles either
uniform or on a displaced lattice with 30 % of them in 200 halos.

A case is a dict of plain values:
  kind      force (sr_force), noalloc (Context.force_noalloc), grad (sr_force
            and its backward), batched (sr_force_batched over the rungs 0..7),
            pm (lr_force), total (p3m_force), step (Context.kdk_step)
  n         particles, any number
  set       uniform or clustered
  precision fp64 or fp32
  layout    auto: a program that only calls the library; tuned: one that
            keeps a handle with the layout the autotuner settles on for sets
            of this size
  masses    per-particle masses (else all ones)
  active    share of the particles that receive (1: all, no mask)
  soft      B-spline softening of 0.03 mean particle distances
  n_grid    PM grid points per dimension (pm, total, step)
"""
from __future__ import annotations

import math

import torch

import paper_2112_01508_amd as p3

N_HALOS, HALO_SHARE = 200, 0.3
RUNGS = list(range(8))
ETA, MAX_RUNG = 0.025, 3


def _case(kind, n, set="clustered", precision="fp32", layout="auto", masses=False, active=1.0,
          soft=False, n_grid=0, name=None):
    c = dict(kind=kind, n=n, set=set, precision=precision, layout=layout, masses=masses,
             active=active, soft=soft, n_grid=n_grid)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a test problem or a notebook: latency of a whole call
        _case("force", 4096, "uniform", "fp64", name="force_4k_fp64"),
        # a serving loop or a captured graph that may not allocate
        _case("noalloc", 32 ** 3, "uniform", "fp32", name="noalloc_32k_fp32"),
        # gradient-based fitting of a small field, in double precision
        _case("grad", 64 ** 3, precision="fp64", masses=True, name="grad_262k_fp64"),
        # the force of one step on a set of ragged size, softened, with masses
        _case("force", 300007, masses=True, soft=True, name="force_300k_soft_fp32"),
        # the force of one production step, layout tuned once per run
        _case("force", 128 ** 3, layout="tuned", name="force_2m_fp32"),
        _case("force", 128 ** 3, precision="fp64", layout="tuned", name="force_2m_fp64"),
        # a kick of the upper rungs: a fifth of the particles receive
        _case("force", 128 ** 3, active=0.2, name="force_2m_masked_fp32"),
        # all kick depths of the rung hierarchy in one launch
        _case("batched", 96 ** 3, layout="tuned", masses=True, name="batched_885k_fp32"),
        # the mesh half alone, at the paper's two cells per particle distance
        _case("pm", 128 ** 3, n_grid=256, name="pm_2m_256"),
        # the whole force of a small box
        _case("total", 64 ** 3, n_grid=128, name="total_262k_fp32"),
        # a synchronised step of the rung-hierarchical integrator
        _case("step", 48 ** 3, precision="fp64", soft=True, n_grid=128, name="step_111k_fp64"),
        # the largest: forward and backward on a set that fills the GPU for long
        _case("grad", 256 ** 3, layout="tuned", name="grad_17m_fp32"),
    ]


# sizes per kind (log-uniform), the smallest and largest a drawn case takes
_RANGE = {"force": (1000, 3_000_000), "noalloc": (1000, 1 << 17), "grad": (8000, 2_000_000),
          "batched": (30_000, 1_000_000), "pm": (1000, 3_000_000), "total": (8000, 2_000_000),
          "step": (8000, 120_000)}


def draw(rng):
    kind = rng.choice(["force", "force", "force", "noalloc", "grad", "grad", "batched", "pm",
                       "total", "step"])
    lo, hi = _RANGE[kind]
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    clustered = n >= 32 ** 3 and rng.random() < 0.8
    layout = "auto"
    if kind in ("force", "grad", "batched") and n >= 64 ** 3 and rng.random() < 0.5:
        layout = "tuned"
    if kind == "batched":
        layout = "tuned"
    precision = rng.choice(["fp64", "fp32"])
    if kind == "pm" or kind == "step":
        precision = "fp64"
    n_grid = 0
    if kind in ("pm", "total", "step"):
        n_grid = min(256, max(32, 1 << round(math.log2(2 * n ** (1 / 3)))))
    return _case(kind, n, "clustered" if clustered else "uniform", precision, layout,
                 masses=rng.random() < 0.4,
                 active=round(rng.uniform(0.05, 0.6), 3)
                 if kind in ("force", "grad") and rng.random() < 0.25 else 1.0,
                 soft=kind == "step" or (kind in ("force", "grad") and rng.random() < 0.25),
                 n_grid=n_grid)


# ---- inputs ---------------------------------------------------------------------


def _scales(n, n_grid=0):
    """x_s and r_cut: mesh cells of half the mean particle distance, or the
    PM grid's own cells where the call has one."""
    cell = 1.0 / n_grid if n_grid else 0.5 / n ** (1 / 3)
    return 1.25 * cell, 5.625 * cell


def _eps(case):
    return 0.03 / case["n"] ** (1 / 3) if case["soft"] else 0.0


def _clustered(n, gen):
    """A displaced lattice (P(k) ~ k^-2, rms half a mesh cell) with 30 % of
    the particles moved into 200 NFW-like halos of 2 to 20 mesh cells."""
    dev, f64 = gen.device, torch.float64
    m = math.ceil(n ** (1 / 3) - 1e-9)
    cell = 0.5 / n ** (1 / 3)
    f = torch.fft.fftfreq(m, d=1.0 / m, device=dev, dtype=f64) * (2 * math.pi)
    fz = torch.fft.rfftfreq(m, d=1.0 / m, device=dev, dtype=f64) * (2 * math.pi)
    dk = torch.fft.rfftn(torch.randn((m, m, m), generator=gen, device=dev, dtype=f64))
    k2 = f[:, None, None] ** 2 + f[None, :, None] ** 2 + fz ** 2
    k2[0, 0, 0] = 1.0
    dk *= k2 ** -1.5
    dk[0, 0, 0] = 0.0
    psi = torch.stack([torch.fft.irfftn(1j * k * dk, s=(m, m, m)).reshape(-1)
                       for k in (f[:, None, None], f[None, :, None], fz)], 1)
    del dk, k2
    psi *= 0.5 * cell / psi.square().sum(1).mean().sqrt()
    q = (torch.arange(m, device=dev, dtype=f64) + 0.5) / m
    pos = torch.cartesian_prod(q, q, q) + psi
    if m ** 3 > n:   # a ragged number: the lattice with sites left out
        pos = pos[torch.randperm(m ** 3, generator=gen, device=dev)[:n].sort().values]
    n_in = int(HALO_SHARE * n)
    u = torch.rand((N_HALOS, 5), generator=gen, device=dev, dtype=f64)
    radius = cell * torch.exp(math.log(2.0) + u[:, 3] * math.log(10.0))
    conc = 5.0 + 10.0 * u[:, 4]
    owner = torch.multinomial(radius ** 3, n_in, replacement=True, generator=gen)
    x = torch.linspace(0.0, 1.0, 2048, device=dev, dtype=f64) ** 2 * conc[:, None]
    enclosed = torch.log1p(x) - x / (1 + x)   # one row per halo
    t = torch.rand(n_in, generator=gen, device=dev, dtype=f64)
    row = enclosed[:, -1:].contiguous()
    # invert the enclosed mass: one sorted table over all halos, owner + fraction
    table = (enclosed / row * (1 - 1e-12)
             + torch.arange(N_HALOS, device=dev, dtype=f64)[:, None]).reshape(-1)
    at = torch.searchsorted(table, owner + t * (1 - 1e-9)).clamp(1, table.numel() - 1)
    lo, hi = table[at - 1], table[at]
    frac = ((owner + t - lo) / (hi - lo).clamp(min=1e-300)).clamp(0, 1)
    xs = x.reshape(-1)
    prev = torch.where(at % 2048 == 0, xs[at], xs[at - 1])
    r = (prev + frac * (xs[at] - prev)) / conc[owner] * radius[owner]
    d = torch.randn((n_in, 3), generator=gen, device=dev, dtype=f64)
    d *= (r / d.square().sum(1).sqrt())[:, None]
    chosen = torch.randperm(n, generator=gen, device=dev)[:n_in]
    pos[chosen] = u[owner, :3] + d
    return pos


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, f64 = case["n"], torch.float64
    if case["set"] == "clustered":
        pos = _clustered(n, gen)
    else:
        pos = torch.rand((n, 3), generator=gen, device="cuda", dtype=f64)
    pos = torch.remainder(pos, 1.0)
    pos = torch.where(pos >= 1.0, torch.zeros_like(pos), pos).contiguous()
    mass = None
    if case["masses"]:
        mass = 0.5 + torch.rand(n, generator=gen, device="cuda", dtype=f64)
    active = None
    if case["active"] < 1.0:
        active = (torch.rand(n, generator=gen, device="cuda") < case["active"]).to(torch.uint8)
    weights = None
    if case["kind"] == "grad":
        weights = torch.randn((n, 3), generator=gen, device="cuda", dtype=f64)
    rung = None
    if case["kind"] == "batched":
        rung = _density_rungs(pos)
    return pos, mass, active, weights, rung


def _density_rungs(pos):
    """clamp(floor(log2(rho / mean) / 1.5), 0, 7) from counts in 27-cell blocks."""
    n = pos.shape[0]
    m = max(4, int(n ** (1 / 3)))
    c = (pos * m).long().clamp(max=m - 1)
    flat = (c[:, 0] * m + c[:, 1]) * m + c[:, 2]
    block = torch.bincount(flat, minlength=m ** 3).double().reshape(m, m, m)
    for axis in range(3):
        block = block.roll(1, axis) + block + block.roll(-1, axis)
    ratio = block.reshape(-1)[flat] * (m ** 3 / (27.0 * n))
    return torch.floor(torch.log2(ratio) / 1.5).clamp(0, 7).to(torch.uint8)


# Handles as a program keeps them: made once, used for every set it works on.
_handles = {}


def _handle(case):
    """None: the library's default handle."""
    layout = None
    if case["layout"] == "tuned":
        target = 4096 if case["n"] >= 1_000_000 or case["kind"] == "batched" else 512
        if case["kind"] == "batched":
            layout = (1, target, 32, 1)
        else:
            layout = (1, target, 32 if case["precision"] == "fp32" else 16, 2)
    # a step sets its own softening
    eps = 0.0 if case["kind"] == "step" else _eps(case)
    if layout is None and eps == 0.0:
        return p3.default_context()
    key = (layout, eps)
    if key not in _handles:
        h = p3.Context()
        if layout:
            h.set_config(*layout)
        h.set_softening(eps)
        _handles[key] = h
    return _handles[key]


def prepare(case, seed):
    pos, mass, active, weights, rung = _inputs(case, seed)
    x_s, r_cut = _scales(case["n"], case["n_grid"])
    state = dict(case=case, handle=_handle(case), pos=pos, mass=mass, active=active,
                 weights=weights, rung=rung,
                 kw=dict(box=1.0, x_s=x_s, r_cut=r_cut, precision=case["precision"]))
    if case["kind"] == "grad":
        pos.requires_grad_(True)
    if case["kind"] == "step":
        state["vel"] = torch.zeros_like(pos)
        state["rung"] = torch.zeros(case["n"], dtype=torch.uint8, device="cuda")
    return state


def _dt(case):
    """A step that leaves most particles of a unit-mass set on rung 0."""
    return 0.5 * math.sqrt(2.0 * ETA * 0.03 / case["n"])


def run(state):
    case, h, kw = state["case"], state["handle"], state["kw"]
    pos, mass, active = state["pos"], state["mass"], state["active"]
    kind = case["kind"]
    if kind == "force":
        return p3.sr_force(pos, mass, active, context=h, **kw)
    if kind == "noalloc":
        return h.force_noalloc(pos, mass, active, **kw)
    if kind == "grad":
        acc = p3.sr_force(pos, mass, active, context=h, **kw)
        (grad,) = torch.autograd.grad(acc, pos, state["weights"])
        return acc.detach(), grad
    if kind == "batched":
        return p3.sr_force_batched(pos, mass, state["rung"], RUNGS, context=h, **kw)
    if kind == "pm":
        return p3.lr_force(pos, mass, active, box=1.0, n_grid=case["n_grid"], x_s=kw["x_s"],
                           context=h)
    if kind == "total":
        return p3.p3m_force(pos, mass, active, n_grid=case["n_grid"], context=h, **kw)
    # the step advances its arguments in place: on copies, so that the state
    # before it stays at hand
    p, v, r = pos.clone(), state["vel"].clone(), state["rung"].clone()
    return h.kdk_step(p, v, mass, r, n_grid=case["n_grid"], dt=_dt(case), eta=ETA,
                      eps=_eps(case), max_rung=MAX_RUNG, **kw)


def work(case):
    """Algorithmic bytes (each input read and each output written once) and
    flops (40 per ordered pair within r_cut, 60 for the adjoint, 5 n log2 n
    per FFT and 200 per particle for the mesh)."""
    n = case["n"]
    volume = 4.0 / 3.0 * math.pi * _scales(n, case["n_grid"])[1] ** 3
    near = n * volume * (1.0 + (7.0 * n / 128 ** 3 if case["set"] == "clustered" else 0.0))
    rows = n * case["active"]
    bytes_ = 24 * n + (8 * n if case["masses"] else 0) + (n if case["active"] < 1 else 0)
    g3 = float(case["n_grid"]) ** 3
    mesh = 2 * 2.5 * g3 * math.log2(max(g3, 2.0)) + 200.0 * n
    kind = case["kind"]
    if kind == "grad":
        return {"bytes": bytes_ + 72 * n, "flops": 100.0 * rows * near}
    if kind == "batched":
        return {"bytes": bytes_ + n + 8 * 24 * n, "flops": 40.0 * 2.5 * n * near}
    if kind == "pm":
        return {"bytes": bytes_ + 24 * n, "flops": mesh}
    if kind == "total":
        return {"bytes": bytes_ + 24 * n, "flops": 40.0 * rows * near + mesh}
    if kind == "step":
        return {"bytes": bytes_ + 75 * n, "flops": 40.0 * 3.0 * n * near + 2 * mesh}
    return {"bytes": bytes_ + 24 * n, "flops": 40.0 * rows * near}


# ---- the same results in 64 bits, from their definitions ----------------------------


def _phi(r, x_s, eps):
    """Pair factor g(u) / r^3, softened inside eps_B = 2.8 eps, and its
    derivative divided by r."""
    u = r / (2.0 * x_s)
    gauss = torch.exp(-u * u)
    g = torch.erfc(u) + 2.0 / math.sqrt(math.pi) * u * gauss
    phi = g / r ** 3
    dphi = -3.0 * g / r ** 5 - gauss / (2.0 * math.sqrt(math.pi) * x_s ** 3 * r * r)
    if eps > 0.0:
        eb = 2.8 * eps
        # (g - 1) / u^3 from its series: eb is well below x_s
        s, ds, t = torch.zeros_like(u), torch.zeros_like(u), u.clamp(max=0.75) ** 2
        for k in range(24, 0, -1):
            c = 2.0 / math.sqrt(math.pi) * (-1) ** k / math.factorial(k) * 2 * k / (2 * k + 1)
            ds = ds * t + s
            s = s * t + c
        x = r / eb
        k3 = 32.0 / eb ** 3
        inner = k3 * (x ** 3 - 1.2 * x * x + 1.0 / 3.0)
        outer = k3 * (-x ** 3 / 3 + 1.2 * x * x - 1.5 * x + 2.0 / 3 - 1 / (480 * x ** 3))
        d_in = k3 / eb * (3 * x * x - 2.4 * x)
        d_out = k3 / eb * (-x * x + 2.4 * x - 1.5 + 3 / (480 * x ** 4))
        soft = s / (2 * x_s) ** 3 + torch.where(x < 0.5, inner, outer)
        # d/dr of s(u^2) / (2 x_s)^3 is ds * 2 u / (2 x_s) / (2 x_s)^3
        dsoft = 2 * ds / (2 * x_s) ** 5 + torch.where(x < 0.5, d_in, d_out) / r
        phi, dphi = torch.where(r < eb, soft, phi), torch.where(r < eb, dsoft, dphi)
    return phi, dphi


def _pairs(pos, r_cut, rows):
    """(i, j, dx) of the ordered pairs within r_cut with i in `rows`, chunk by
    chunk, from cells of side >= r_cut."""
    n, dev = pos.shape[0], pos.device
    m = max(3, int(1.0 / (r_cut * (1 + 1e-9))))
    c = (pos * m).long().clamp(max=m - 1)
    order = torch.argsort((c[:, 0] * m + c[:, 1]) * m + c[:, 2])
    p = pos[order]
    flat = ((c[:, 0] * m + c[:, 1]) * m + c[:, 2])[order]
    start = torch.searchsorted(flat, torch.arange(m ** 3 + 1, device=dev))
    for ox in (-1, 0, 1):
        for oy in (-1, 0, 1):
            for oz in (-1, 0, 1):
                nb = (c[rows] + torch.tensor([ox, oy, oz], device=dev)) % m
                nb = (nb[:, 0] * m + nb[:, 1]) * m + nb[:, 2]
                a, length = start[nb], start[nb + 1] - start[nb]
                end = torch.cumsum(length, 0)
                total = int(end[-1]) if end.numel() else 0
                cuts = torch.searchsorted(end, torch.arange(0, total, 1 << 25, device=dev),
                                          right=True).tolist() + [rows.numel()]
                for b, e in zip(cuts[:-1], cuts[1:]):
                    ln = length[b:e]
                    row = torch.repeat_interleave(torch.arange(b, e, device=dev), ln)
                    if row.numel() == 0:
                        continue
                    off = torch.arange(row.numel(), device=dev) - (torch.cumsum(ln, 0) - ln)[row - b]
                    j = a[row] + off
                    i = rows[row]
                    d = pos[i] - p[j]
                    d -= torch.round(d)
                    r2 = d.square().sum(1)
                    keep = torch.nonzero((r2 < r_cut * r_cut) & (r2 > 0)).squeeze(1)
                    yield i[keep], order[j[keep]], d[keep], r2[keep].sqrt()


def _short(pos, mass, rows, x_s, r_cut, eps):
    acc = torch.zeros_like(pos)
    for i, j, d, r in _pairs(pos, r_cut, rows):
        f = _phi(r, x_s, eps)[0]
        if mass is not None:
            f = f * mass[j]
        acc.index_add_(0, i, d * -f[:, None])
    return acc


def _short_vjp(pos, mass, active, w, x_s, r_cut, eps):
    w = w if active is None else w * active[:, None]
    out = torch.zeros_like(pos)
    for i, j, d, r in _pairs(pos, r_cut, torch.arange(pos.shape[0], device=pos.device)):
        phi, dphi = _phi(r, x_s, eps)
        if mass is None:
            v = w[i] - w[j]
        else:
            v = mass[j, None] * w[i] - mass[i, None] * w[j]
        out.index_add_(0, i, -(phi[:, None] * v + (dphi * (d * v).sum(1))[:, None] * d))
    return out


def _cic(pos, n_grid):
    u = pos * n_grid - 0.5
    lo = torch.floor(u)
    f = u - lo
    lo = lo.long()
    for k in range(8):
        bit = torch.tensor([k >> 2 & 1, k >> 1 & 1, k & 1], device=pos.device)
        at = (lo + bit) % n_grid
        w = torch.where(bit.bool(), f, 1.0 - f).prod(1)
        yield (at[:, 0] * n_grid + at[:, 1]) * n_grid + at[:, 2], w


def _long(pos, mass, n_grid, x_s):
    dev, f64 = pos.device, torch.float64
    rho = torch.zeros(n_grid ** 3, device=dev, dtype=f64)
    for at, w in _cic(pos, n_grid):
        rho.index_add_(0, at, w if mass is None else w * mass)
    h = torch.fft.fftfreq(n_grid, d=1.0 / n_grid, device=dev, dtype=f64)
    s = torch.sinc(h / n_grid)
    k2 = (2 * math.pi) ** 2 * (h[:, None, None] ** 2 + h[:, None] ** 2 + h ** 2)
    k2[0, 0, 0] = 1.0
    green = torch.exp(-x_s * x_s * k2) / k2 / (s[:, None, None] * s[:, None] * s) ** 4
    green[0, 0, 0] = 0.0
    phi = torch.fft.ifftn(green * torch.fft.fftn(rho.reshape((n_grid,) * 3))).real
    acc = torch.zeros_like(pos)
    for axis in range(3):
        diff = (phi.roll(2, axis) - 8 * phi.roll(1, axis) + 8 * phi.roll(-1, axis)
                - phi.roll(-2, axis)).reshape(-1) / 12.0
        for at, w in _cic(pos, n_grid):
            acc[:, axis] += w * diff[at]
    return acc * (4.0 * math.pi * n_grid ** 4)


def _rung_of(acc, dt, eps):
    z = dt * torch.sqrt(acc.square().sum(1).sqrt() / (2.0 * ETA * eps))
    return torch.ceil(torch.log2(z.clamp(min=1e-300))).clamp(0, MAX_RUNG).long()


def _step(pos, mass, case, x_s, r_cut):
    """One synchronised step: rung l kicks every dt / 2^l, positions drift in
    dt / 2^L, times in units of dt / 2^(L + 1)."""
    eps, dt, n = _eps(case), _dt(case), case["n"]
    x, v = pos.clone(), torch.zeros_like(pos)
    acc = _short(x, mass, torch.arange(n, device=x.device), x_s, r_cut, eps)
    rung = _rung_of(acc, dt, eps)
    top = int(rung.max())
    half, period = dt / 2 ** (top + 1), 2 ** (top + 1)
    span = period >> rung
    t_q, t_next = span // 2, span.clone()
    v += acc * (t_q.double() * half)[:, None]
    v += _long(x, mass, case["n_grid"], x_s) * (period // 2 * half)
    last = torch.zeros_like(x)
    for t in range(2, period + 1, 2):
        x = torch.remainder(x + v * (2 * half), 1.0)
        x = torch.where(x >= 1.0, x - 1.0, x)
        due = torch.nonzero(t_next == t).squeeze(1)
        if due.numel():
            a = _short(x, mass, due, x_s, r_cut, eps)[due]
            last[due] = a
            span = period >> rung[due]
            target = torch.full_like(due, period) if t == period else t + span // 2
            v[due] += a * ((target - t_q[due]).double() * half)[:, None]
            t_q[due] = target
            if t < period:
                want, l = _rung_of(a, dt, eps).clamp(max=top), rung[due]
                down = (want < l) & ((t + span) % (2 * span) == 0)
                l = l + (want > l).long() - down.long()
                rung[due] = l
                span = period >> l
                t_next[due] = (t // span + 1) * span
    v += _long(x, mass, case["n_grid"], x_s) * (period // 2 * half)
    return x, v, _rung_of(last, dt, eps).to(torch.uint8)


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if n > 3_000_000:   # over 1e10 pairs
        return None
    pos, mass, active, weights, rung = _inputs(case, seed)
    x_s, r_cut = _scales(n, case["n_grid"])
    eps = _eps(case)
    if kind == "pm":
        acc = _long(pos, mass, case["n_grid"], x_s)
        return acc if active is None else acc * active[:, None]
    if kind == "step":
        return _step(pos, mass, case, x_s, r_cut)
    rows = torch.arange(n, device=pos.device)
    if active is not None:
        rows = rows[active.bool()]
    if kind == "batched":
        acc = _short(pos, mass, rows, x_s, r_cut, eps)
        return torch.stack([acc * (rung >= k)[:, None] for k in RUNGS])
    acc = _short(pos, mass, rows, x_s, r_cut, eps)
    if kind == "total":
        acc += _long(pos, mass, case["n_grid"], x_s)
    if kind == "grad":
        return acc, _short_vjp(pos, mass, active, weights, x_s, r_cut, eps)
    return acc
