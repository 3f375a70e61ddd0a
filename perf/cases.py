"""The work that a user of this framework has it do, as cases that can be timed and checked.

A case is one pass through the public entry points (`grpic.Context`, `adjoint.FrozenFieldPush`) on
inputs made from a seed:

  steps    a run of full PIC steps from a checkpoint, as a simulation goes between two of its cell
           sorts: the checkpoint's fields are restored, the particles are sorted into the working
           set (or copied there), then `steps` steps; with `ranked` the last step's fused pass ranks
           for a closing sort
  frozen   test particles in a frozen field (adjoint.FrozenFieldPush), the forward run and, with
           `grad`, its backward sweep
  fields   the field stages alone with given currents
  inject   the cell sort and pair injection into the slots behind the live ones
  diag     diagnostics with the per-particle energies and the Gauss residual

`exact` holds a plain torch FP64 statement of the same mathematics, written from the equations.
"""
from __future__ import annotations

import math

import torch

from paper_2511_17701_amd import adjoint, grpic

DEV = "cuda"
KAPPA = 1e-7  # deposited charge per unit weight: dense enough for the currents to show in the fields


# ------------------------------------------------------------------------------------- the cases
def _steps(name, n_r, n_th, **kw):
    """Defaults of a `steps` case: Kerr a = 0.9, Wald field, 16 particles per cell, fused passes."""
    c = dict(name=name, kind="steps", n_r=n_r, n_th=n_th, a=0.9, r_in=0.0, r_max=50.0, B0=1.0, T=1.0, ppc=16, pairs=0,
             geo=0, form="fp64", init="wald", n_filter=0, n_absorb=0, r0=0.0, h0=0.0, steps=10, fused=True, sort=True,
             ranked=False)
    c.update(kw)
    return c


def listed():
    return [
        # a few thousand particles on a coarse grid: every launch is short, so latency and launches count
        _steps("tiny_fp32", 40, 56, a=0.9, r_max=20.0, ppc=0, pairs=1500, form="fp32", n_filter=2, n_absorb=4, sort=False),
        # the 64^2 configuration (1e5 cold particles) through Context.step's default, push and deposit apart
        _steps("c1_64_unfused", 64, 64, r_max=20.0, T=0.1, ppc=0, pairs=50_000, fused=False, sort=False),
        # the 512^2 configuration with its neutral geodesics: an ordinary double-precision run
        _steps("c2_512_fp64", 512, 512, geo=1000),
        # the 2048^2 configuration in single precision: an ordinary large run
        _steps("c3_2048_fp32", 2048, 2048, a=0.99, r_max=100.0, B0=10.0, ppc=32, form="fp32"),
        # the benchmark's default workload, the largest: 4096^2, filter passes, absorbing layer
        _steps("c5_4096_fp32", 4096, 4096, a=0.95, r_max=200.0, B0=10.0, form="fp32", n_filter=4, n_absorb=32),
        # the BZ-monopole shape (90 per cell) at a quarter of its cells, closed by the ranked sort as the benchmark does
        _steps("c6_monopole_fp64", 1024, 1024, a=0.2, r_in=1.0, r_max=10.0, T=0.5, ppc=90, init="monopole", n_absorb=47,
               ranked=True, sort=False),
        # the general quasi-spherical map on a ragged grid, push and deposit apart, an odd number of filter passes
        _steps("c7_qks_ragged", 701, 533, a=0.2, r_in=1.0, r_max=10.0, T=0.5, ppc=24, init="monopole", n_filter=5,
               n_absorb=33, r0=0.5, h0=0.3, fused=False),
        # test particles: a thousand, forward and gradient (an optimiser's inner call)
        dict(name="frozen_1k_grad", kind="frozen", n_r=64, n_th=64, a=0.9, r_max=20.0, B0=1.0, T=0.1, pairs=509, steps=5,
             n_iter=200, init="wald", grad=True),
        # the 256^2 differentiation configuration, 1e6 particles
        dict(name="frozen_c4_grad", kind="frozen", n_r=256, n_th=256, a=0.9, r_max=20.0, B0=1.0, T=1.0, pairs=500_000,
             steps=20, n_iter=200, init="wald", grad=True),
        # the field solver alone in double precision, ragged, with filter passes and the absorbing layer
        dict(name="fields_1537_fp64", kind="fields", n_r=1537, n_th=1023, a=0.9, r_max=50.0, B0=1.0, form="fp64",
             n_filter=3, n_absorb=20, steps=5),
        # sort and pair injection every few steps of a magnetosphere run
        dict(name="inject_1500_fp32", kind="inject", n_r=1500, n_th=1100, a=0.2, r_in=1.0, r_max=12.0, B0=1.0, T=0.5,
             ppc=24, form="fp32", init="monopole"),
        # an output step: energies, angular momenta and the Gauss residual
        dict(name="diag_2048_fp32", kind="diag", n_r=2048, n_th=1536, a=0.95, r_max=100.0, B0=1.0, T=1.0, ppc=16,
             form="fp32", n_filter=2, n_absorb=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, sizes spread over the listed range (ragged grids, odd counts)."""
    kind = rng.choice(["steps", "steps", "steps", "steps", "frozen", "fields", "inject", "diag"])
    a, r_max = rng.uniform(0.0, 0.99), rng.uniform(16.0, 200.0)
    mono = rng.random() < 0.3
    init, form = ("monopole" if mono else "wald"), rng.choice(["fp32", "fp64"])
    B0, T = rng.choice([1.0, 10.0]), rng.choice([0.1, 0.5, 1.0])
    if kind == "frozen":
        n = _log(rng, 24, 400)
        return dict(kind=kind, n_r=n, n_th=_log(rng, 24, 400), a=a, r_max=20.0, B0=B0, T=T, pairs=_log(rng, 100, 400_000),
                    steps=rng.randint(3, 20), n_iter=200, init=init, grad=rng.random() < 0.7)
    n_r = _log(rng, 24, 2500)
    n_th = max(24, min(2500, int(n_r * math.exp(rng.uniform(-0.7, 0.7)))))
    n_f = rng.choice([0, 0, 1, 2, 4, 7])
    n_a = rng.choice([0, max(2, n_r // 40)])
    ppc = 2 * rng.randint(2, 24)
    while n_r * n_th * ppc > 100_000_000:
        ppc = max(2, 2 * (ppc // 4))
    if kind == "fields":
        return dict(kind=kind, n_r=n_r, n_th=n_th, a=a, r_max=r_max, B0=B0, form=form, n_filter=n_f, n_absorb=n_a,
                    steps=rng.randint(1, 10))
    if kind == "inject":
        return dict(kind=kind, n_r=n_r, n_th=n_th, a=0.2, r_in=1.0, r_max=rng.uniform(8.0, 20.0), B0=1.0, T=0.5, ppc=ppc,
                    form=form, init="monopole")
    if kind == "diag":
        return dict(kind=kind, n_r=n_r, n_th=n_th, a=a, r_max=r_max, B0=B0, T=T, ppc=ppc, form=form, n_filter=n_f,
                    n_absorb=n_a)
    c = _steps("", n_r, n_th, a=a, r_max=r_max, B0=B0, T=T, form=form, init=init, n_filter=n_f, n_absorb=n_a, ppc=ppc)
    del c["name"]
    if rng.random() < 0.25:
        c.update(ppc=0, pairs=_log(rng, 500, 500_000) + 1)
    if rng.random() < 0.25:
        c.update(r0=0.3, h0=rng.choice([0.3, -0.2]))
    c["geo"] = rng.choice([0, 0, 333]) if c["r0"] == 0.0 else 0
    c["fused"] = rng.random() < 0.75
    c["ranked"] = c["fused"] and rng.random() < 0.3
    c["sort"] = not c["ranked"] and rng.random() < 0.7
    c["steps"] = rng.choice([1, 2, 4, 8, 12])
    return c


# ------------------------------------------------------------------------------------ preparation
def _r_in(c):
    return c.get("r_in", 0.0) or 0.9 * (1.0 + math.sqrt(1.0 - c["a"] ** 2))


def _fp32(c):
    return c.get("form") == "fp32"


def _context(c):
    return grpic.Context(c["a"], 1.0, _r_in(c), c["r_max"], c["n_r"], c["n_th"], cfl=0.5, n_iter=c.get("n_iter", 10),
                         charge_scale=KAPPA, n_filter=c.get("n_filter", 0), n_absorb=c.get("n_absorb", 0),
                         r0=c.get("r0", 0.0), h0=c.get("h0", 0.0),
                         precision=grpic.GRPIC_FP32 if _fp32(c) else grpic.GRPIC_FP64)


def _set(ctx, n):
    """A particle set in one allocation (its arrays are views), so that a checkpoint is one copy."""
    item = {"tag": 1, **{k: 4 for k in grpic.INT_FIELDS}}
    size = [item.get(k, torch.empty((), dtype=ctx.dtype).element_size()) for k in grpic.PARTICLE_FIELDS]
    at, total = [], 0
    for s in size:
        at.append(total)
        total += -(-n * s // 256) * 256
    buf = torch.zeros(total, dtype=torch.uint8, device=DEV)
    P = {}
    for k, s, o in zip(grpic.PARTICLE_FIELDS, size, at):
        dt = torch.uint8 if k == "tag" else torch.int32 if k in grpic.INT_FIELDS else ctx.dtype
        P[k] = buf[o:o + n * s].view(dt)
    return buf, P


def _wander(c, P, n, gen, sort_interval=10):
    """Displaces the particles as a sort interval does (a cell or a few next to the hole, a fraction
    of one far out), so that the slots are in the order that the passes meet between two sorts; the
    previous position is where each was a tenth of that before."""
    xi = math.log((c["r_max"] - c.get("r0", 0.0)) / (_r_in(c) - c.get("r0", 0.0))) / c["n_r"]
    reach = 0.25 * sort_interval * torch.exp(-xi * (P["i1"][:n].double() + P["dx1"][:n].double()))
    for q, hi in (("1", c["n_r"]), ("2", c["n_th"])):
        i, dx = P["i" + q], P["dx" + q]
        x = i[:n].double() + dx[:n].double()
        x += reach * torch.randn(n, dtype=torch.float64, device=DEV, generator=gen)
        x = x.abs()
        x = torch.where(x > hi, 2.0 * hi - x, x).clamp(0.0, hi * (1.0 - 1e-12))
        f = x.floor().clamp(max=hi - 1)
        i[:n] = f.int()
        dx[:n] = (x - f).to(dx.dtype)
        y = (x - (0.1 * reach)).clamp(min=0.0)
        f = y.floor().clamp(max=hi - 1)
        P["i" + q + "p"][:n] = f.int()
        P["dx" + q + "p"][:n] = (y - f).to(dx.dtype)


def _fields(c, ctx, B0):
    F = ctx.new_fields(DEV)
    (ctx.fields_init_monopole if c.get("init") == "monopole" else ctx.fields_init_wald)(F, B0)
    return F


def _count(c):
    return c["n_r"] * c["n_th"] * c["ppc"] if c.get("ppc", 0) else 2 * c["pairs"]


def prepare(case, seed):
    c = case
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    B0 = c["B0"] * (1.0 + 0.1 * torch.rand((), dtype=torch.float64, device=DEV, generator=gen).item())
    ctx = _context(c)
    s = dict(case=c, ctx=ctx, B0=B0)
    if c["kind"] == "fields":
        s["F0"] = _fields(c, ctx, B0)
        J = grpic.PLANES["J"]
        s["F0"][J:J + 3] = 1e-6 * torch.randn((3,) + tuple(ctx.shape), dtype=ctx.dtype, device=DEV, generator=gen)
        s["F"] = s["F0"].clone()
        return s
    n, geo = _count(c), c.get("geo", 0)
    if c["kind"] == "frozen":
        P = ctx.new_particles(n, DEV)
        ctx.particles_init(P, c["pairs"], 0, c["T"], 0, int(seed))
        s["start"] = P
        s["u0"] = torch.stack([P["u1"], P["u2"], P["u3"]], 1).requires_grad_(c["grad"])
        s["amplitude"] = torch.tensor(B0, dtype=torch.float64, requires_grad=c["grad"])
        s["run"] = adjoint.FrozenRun(ctx, P, c["steps"], init=c["init"])
        s["g"] = torch.randn((n, 5), dtype=torch.float64, device=DEV, generator=gen)
        return s
    room = n // 4 if c["kind"] == "inject" else 0  # free slots for the injected pairs
    s["buf0"], s["P0"] = _set(ctx, n + geo + room)
    loaded = {k: v[:n + geo] for k, v in s["P0"].items()}
    ctx.particles_init(loaded, c.get("pairs", 0), c.get("ppc", 0), c["T"], geo, int(seed))
    _wander(c, s["P0"], n, gen, 10 if c.get("sort", True) else 2)
    s["F0"] = _fields(c, ctx, B0)
    if c["kind"] == "diag":
        return s
    s["buf"], s["P"] = _set(ctx, n + geo + room)
    if c["kind"] == "inject":
        s["seed"] = int(seed)
        return s
    s["F"] = s["F0"].clone()
    if c["ranked"]:
        s["Q"] = _set(ctx, n + geo)[1]
    return s


# ------------------------------------------------------------------------------------------- runs
def _planes(c, F):
    """The time-advanced planes D, B, D0, B0 (the others are scratch or targets), and in double precision the
    last step's current: the zigzag current of a particle that ends a step within a rounding of a cell face
    jumps from one cell to the next, which a single-precision run of many particles always meets somewhere."""
    return {"em": F[0:12]} if _fp32(c) else {"em": F[0:12], "J0": F[21:24]}


def _particles(c, P):
    """Positions, the conserved u3 and phi; u1, u2 of runs of a step or two (beyond that the particles that pass
    next to an axis amplify a rounding by orders of magnitude)."""
    out = {k: P[k] for k in (("u1", "u2") if c["steps"] <= 2 else ()) + ("u3", "phi")}
    out["x1"], out["x2"] = P["i1"] + P["dx1"], P["i2"] + P["dx2"]
    return out


def _run_steps(s):
    c, ctx, F, P = s["case"], s["ctx"], s["F"], s["P"]
    F.copy_(s["F0"])
    if c["sort"]:
        ctx.sort(s["P0"], P)
    else:
        s["buf"].copy_(s["buf0"])
    for _ in range(c["steps"] - (1 if c["ranked"] else 0)):
        ctx.step(F, P, fused=c["fused"])
    if c["ranked"]:
        ctx.field_advance(F, grpic.PRE_PUSH)
        ctx.push_deposit(F, P, ranked=True)
        ctx.field_advance(F, grpic.POST_DEPOSIT)
        ctx.sort(P, s["Q"], ranked=True)
    out = _planes(c, F)
    # after a sort the order of the particles within a cell is unspecified: their arrays cannot be compared slot by slot
    return out if c["sort"] or c["ranked"] else {**out, **_particles(c, P)}


def run(state):
    s = state
    c, ctx = s["case"], s["ctx"]
    if c["kind"] == "steps":
        return _run_steps(s)
    if c["kind"] == "fields":
        s["F"].copy_(s["F0"])
        for _ in range(c["steps"]):
            ctx.field_advance(s["F"], grpic.PRE_PUSH)
            ctx.field_advance(s["F"], grpic.POST_DEPOSIT)
        return _planes(c, s["F"])
    if c["kind"] == "frozen":
        if not c["grad"]:
            with torch.no_grad():
                return {"final": adjoint.FrozenFieldPush.apply(s["u0"], s["amplitude"], s["run"])}
        final = adjoint.FrozenFieldPush.apply(s["u0"], s["amplitude"], s["run"])
        gu, gB = torch.autograd.grad(final, (s["u0"], s["amplitude"]), s["g"])
        return {"final": final.detach(), "g_u0": gu, "g_B0": gB}
    if c["kind"] == "inject":
        Q = s["P"]
        live = ctx.sort(s["P0"], Q, count=True)
        n = ctx.inject_pairs(s["F0"], Q, 1000.0, c["T"], 1, 1.0, 0, c["n_r"], s["seed"], 0, live)
        new = {k: Q[k][live:live + 2 * n] for k in ("dx1", "dx2", "u1", "u2", "u3")}
        # the sorted slots' cells and weights (the order of the particles within a cell is unspecified)
        return {"live": live, "n": n, **{k: Q[k] for k in ("i1", "i2", "w")}, "new": new}
    return ctx.diagnostics(s["F0"], s["P0"], s["B0"], per_particle=True, gauss_plane=True)


def work(case):
    """Bytes and operations of one pass: every particle's and plane's values read and written once per step."""
    c = case
    real = 4 if _fp32(c) else 8
    cells = (c["n_r"] + 4) * (c["n_th"] + 4)
    if c["kind"] == "fields":
        # per step: D, B, D0, B0, J, J0 in and out
        return {"bytes": c["steps"] * cells * real * 36, "flops": c["steps"] * cells * 400}
    n = _count(c) + c.get("geo", 0)
    part_in, part_out = 9 + 7 * real, 8 + 6 * real + 1  # tag, cell, offsets, u, w, phi | cell, offsets, u, phi, tag
    if c["kind"] == "steps":
        moved = 2 * (9 + 7 * real) * n  # the sort or the restored checkpoint
        return {"bytes": moved + c["steps"] * (n * (part_in + part_out) + cells * real * 36),
                "flops": c["steps"] * (700 * n + 400 * cells)}
    if c["kind"] == "frozen":
        # forward steps; the backward sweep reads each step's state and carries the cotangent
        back = c["steps"] * n * (49 + 80 + 16) if c["grad"] else 0
        return {"bytes": c["steps"] * n * (part_in + part_out) + back, "flops": c["steps"] * n * (600 + (2400 if c["grad"] else 0))}
    if c["kind"] == "inject":
        return {"bytes": n * 2 * (9 + 7 * real) + cells * (3 * real + 8), "flops": 60 * cells}
    return {"bytes": n * (1 + 16 + 8 * real + 2 * real) + cells * 4 * real, "flops": 150 * n + 100 * cells}


# ------------------------------------------------------------------------------------------ exact
class _Exact:
    """The method in plain torch, FP64: the Kerr-Schild 3+1 geometry on the code coordinates, the particle
    step, the zigzag deposit and the field stages, vectorised over particles and planes."""

    def __init__(self, c, dt):
        self.c, self.dt, self.a, self.kappa = c, dt, c["a"], KAPPA
        self.n_r, self.n_th = c["n_r"], c["n_th"]
        self.r0, self.h0 = c.get("r0", 0.0), c.get("h0", 0.0)
        self.xi0 = math.log(_r_in(c) - self.r0)
        self.dxi = math.log((c["r_max"] - self.r0) / (_r_in(c) - self.r0)) / self.n_r
        self.dth = math.pi / self.n_th
        self.n_f, self.n_a, self.n_iter = c.get("n_filter", 0), c.get("n_absorb", 0), c.get("n_iter", 10)

    # geometry
    def at(self, x1, x2, clamp):
        """r, dr/dx1, sin, cos, dtheta/dx2 (mirrored past either axis); clamp: keep 1e-5 rad from the axes."""
        e = torch.exp(self.xi0 + x1 * self.dxi)
        low, high = x2 < 0, x2 > self.n_th
        y = torch.where(low, -x2, torch.where(high, 2.0 * self.n_th - x2, x2))
        # measured from the nearer axis, where sin keeps its relative precision
        far = 2 * y > self.n_th
        eta = torch.where(far, self.n_th - y, y) * self.dth
        p = math.pi
        th = eta + 2 * self.h0 * eta * (p - 2 * eta) * (p - eta) / p ** 2
        T = self.dth * (1 + 2 * self.h0 + 12 * self.h0 * eta * (eta - p) / p ** 2)
        if clamp:  # the derivatives are those of the metric at the clamped angle
            th = torch.where((th < 1e-5) | low | high, th + (1e-5 - th).detach(), th)
        s, co = torch.sin(th), torch.cos(th)
        co = torch.where(far, -co, co)
        s = torch.where(low | high, -s, s) if not clamp else s
        return self.r0 + e, self.dxi * e, s, co, T

    def upper(self, x1, x2):
        """alpha, beta^1, h^11, h^22, h^33, h^13 (theta clamped)."""
        r, R, s, co, T = self.at(x1, x2, True)
        a = self.a
        Sg = r * r + (a * co) ** 2
        S2, ra = Sg + 2 * r, r * r + a * a
        A = ra * ra - a * a * (ra - 2 * r) * s * s
        return (torch.sqrt(Sg / S2), 2 * r / (S2 * R), A / (Sg * S2 * R * R), 1 / (Sg * T * T), 1 / (Sg * s * s), a / (Sg * R))

    def lower(self, i, o1, j, o2):
        """The solver's metric at the grid points (i + o1/2, j + o2/2)."""
        r, R, s, co, T = self.at(i + 0.5 * o1, j + 0.5 * o2, False)
        a = self.a
        Sg = r * r + (a * co) ** 2
        S2, ra = Sg + 2 * r, r * r + a * a
        A = ra * ra - a * a * (ra - 2 * r) * s * s
        al = torch.sqrt(Sg / S2)
        sht = R * T * Sg / al  # sqrt(h) / sin
        h33, h13, h11 = A * s * s / Sg, -a * S2 / Sg * s * s * R, S2 / Sg * R * R
        return dict(al=al, h11=h11, h22=Sg * T * T, h33=h33, w13=sht * h13, wb=sht * sht * s * (2 * r / (S2 * R)), sht=sht, sh=sht * s)

    # particles
    @staticmethod
    def gather(F, i1, d1, i2, d2, h1, h2):
        k1, w1, k2, w2 = i1, d1, i2, d2
        if h1:
            up = d1 >= 0.5
            k1, w1 = torch.where(up, i1, i1 - 1), torch.where(up, d1 - 0.5, d1 + 0.5)
        if h2:
            up = d2 >= 0.5
            k2, w2 = torch.where(up, i2, i2 - 1), torch.where(up, d2 - 0.5, d2 + 0.5)
        k1, k2 = k1 + 2, k2 + 2
        f0 = F[k1, k2] + w2 * (F[k1, k2 + 1] - F[k1, k2])
        f1 = F[k1 + 1, k2] + w2 * (F[k1 + 1, k2 + 1] - F[k1 + 1, k2])
        return f0 + w1 * (f1 - f0)

    def push(self, P, D, B):
        """One update of every moving particle of P (a dict of FP64 / int64 tensors, slots in place)."""
        dt, tag = self.dt, P["tag"]
        gone = (tag & 0x80) != 0
        on = (tag != 0) & ~gone & ((tag & 0x40) == 0)
        i1, i2, d1, d2 = (P[k][on] for k in ("i1", "i2", "dx1", "dx2"))
        u1, u2, u3 = (P[k][on] for k in ("u1", "u2", "u3"))
        t = tag[on]
        q = torch.where((t & 3) == 1, 1.0, torch.where((t & 3) == 2, -1.0, 0.0)).double()
        x1, x2 = (i1 + d1).requires_grad_(True), (i2 + d2).requires_grad_(True)
        m = self.upper(x1, x2)
        g = [torch.autograd.grad(v.sum(), (x1, x2), retain_graph=True) for v in m]
        x1, x2 = x1.detach(), x2.detach()
        al, b1, h11, h22, h33, h13 = (v.detach() for v in m)
        gal, gb1, g11, g22, g33, g13 = g
        low33 = h11 / (h11 * h33 - h13 * h13)
        e1, e2, e3, k13 = torch.sqrt(h11), torch.sqrt(1 / h22), torch.sqrt(low33), -h13 / h11

        def field(X, st):
            v = [self.gather(X[k], i1, d1, i2, d2, *st[k]) for k in range(3)]
            return al * v[0] / e1, al * e2 * v[1], al * e3 * (k13 * v[0] + v[2])
        E, Bh = field(D, ((1, 0), (0, 1), (0, 0))), field(B, ((0, 1), (1, 0), (1, 1)))
        k = 0.25 * q * dt

        def em(u1, u2, u3):
            m = [e1 * (u1 - k13 * u3) + k * E[0], u2 / e2 + k * E[1], u3 / e3 + k * E[2]]
            ig = k / torch.sqrt(1 + m[0] ** 2 + m[1] ** 2 + m[2] ** 2)
            t = [b * ig for b in Bh]
            f = 2 / (1 + t[0] ** 2 + t[1] ** 2 + t[2] ** 2)
            cross = lambda v, w: [v[1] * w[2] - v[2] * w[1], v[2] * w[0] - v[0] * w[2], v[0] * w[1] - v[1] * w[0]]  # noqa: E731
            p = [v + w for v, w in zip(m, cross(m, t))]
            o = [v + f * w + k * y for v, w, y in zip(m, cross(p, t), E)]
            return o[0] / e1 + k13 * e3 * o[2], e2 * o[1], e3 * o[2]
        charged = q != 0
        pick = lambda new, old: [torch.where(charged, v, w) for v, w in zip(new, old)]  # noqa: E731
        u1, u2, u3 = pick(em(u1, u2, u3), (u1, u2, u3))
        mass = torch.where((t & 7) == 7, 0.0, 1.0).double()
        s1, s2 = u1, u2
        for _ in range(self.n_iter):
            b, c = 0.5 * (s1 + u1), 0.5 * (s2 + u2)
            ga = torch.sqrt(mass + h11 * b * b + h22 * c * c + h33 * u3 * u3 + 2 * h13 * b * u3)
            n = [s + dt * (-ga * gal[k] + b * gb1[k] - 0.5 * al / ga * (g11[k] * b * b + g22[k] * c * c + g33[k] * u3 * u3 + 2 * g13[k] * b * u3))
                 for k, s in enumerate((s1, s2))]
            same = bool(((n[0] == u1) & (n[1] == u2)).all())
            u1, u2 = n
            if same:
                break
        u1, u2, u3 = pick(em(u1, u2, u3), (u1, u2, u3))
        v1 = v2 = torch.zeros_like(x1)

        def velocity(m):
            al, b1, h11, h22, h33, h13 = m
            iu = al / torch.sqrt(mass + h11 * u1 * u1 + h22 * u2 * u2 + h33 * u3 * u3 + 2 * h13 * u1 * u3)
            return (h11 * u1 + h13 * u3) * iu - b1, h22 * u2 * iu, (h13 * u1 + h33 * u3) * iu
        for _ in range(self.n_iter):
            n = velocity(self.upper(x1 + 0.5 * v1, x2 + 0.5 * v2))
            n = (dt * n[0], dt * n[1])
            same = bool(((n[0] == v1) & (n[1] == v2)).all())
            v1, v2 = n
            if same:
                break
        w3 = velocity(self.upper(x1 + 0.5 * v1, x2 + 0.5 * v2))[2]
        move = dict(i1=i1, d1=d1, i2=i2, d2=d2, q=q * self.kappa * P["w"][on])
        P["phi"][on] += dt * w3
        y1, y2 = d1 + v1, d2 + v2
        j1, j2 = i1 + y1.floor().long(), i2 + y2.floor().long()
        y1, y2 = y1 - y1.floor(), y2 - y2.floor()
        under, over = j2 < 0, j2 >= self.n_th
        back = under | over
        j2 = torch.where(under, 0, torch.where(over, self.n_th - 1, j2))
        y2, u2 = torch.where(back, 1 - y2, y2), torch.where(back, -u2, u2)
        # a reflected path ends at the reflected position: the deposit takes its own midpoint
        r3 = velocity(self.upper(0.5 * (i1 + d1 + j1 + y1), 0.5 * (i2 + d2 + j2 + y2)))[2]
        move.update(j1=j1, y1=y1, j2=j2, y2=y2, v3=torch.where(back, r3, w3))
        out = (j1 < 0) | (j1 >= self.n_r)
        for key, v in (("i1", j1), ("i2", j2), ("dx1", y1), ("dx2", y2), ("u1", u1), ("u2", u2), ("u3", u3), ("tag", torch.where(out, t | 0x80, t))):
            P[key][on] = v
        P["tag"][gone] = 0
        return move

    def deposit(self, J, m):
        on = m["q"] != 0
        m = {k: v[on] for k, v in m.items()}
        i, j, q, qdt = m["i1"], m["i2"], m["q"], m["q"] / self.dt
        xa, ya = m["d1"], m["d2"]
        di, dj = m["j1"] - i, m["j2"] - j
        xb, yb = di + m["y1"], dj + m["y2"]
        relay = lambda d, s: torch.minimum(d.clamp(max=0) + 1.0, torch.maximum(d.clamp(min=0) + 0.0, s))  # noqa: E731
        xr, yr = relay(di, 0.5 * (xa + xb)), relay(dj, 0.5 * (ya + yb))

        def add(k, ii, jj, v):
            edge = (jj == 0) | (jj == self.n_th)
            v = torch.where(edge, 2 * v, v) if k == 0 else torch.where(edge, 0 * v, v) if k == 2 else v
            J[k].view(-1).index_add_(0, (ii + 2) * (self.n_th + 4) + jj + 2, v)
        for ii, jj, x0, y0, x, y, ox, oy in ((i, j, xa, ya, xr, yr, 0, 0), (i + di, j + dj, xr, yr, xb, yb, di, dj)):
            wx, wy = 0.5 * (x0 + x) - ox, 0.5 * (y0 + y) - oy
            f, g = qdt * (x - x0), qdt * (y - y0)
            add(0, ii, jj, f * (1 - wy))
            add(0, ii, jj + 1, f * wy)
            add(1, ii, jj, g * (1 - wx))
            add(1, ii + 1, jj, g * wx)
        xm, ym = 0.5 * (xa + xb), 0.5 * (ya + yb)
        k, ll = xm.floor(), ym.floor()
        wx, wy, c3 = xm - k, ym - ll, q * m["v3"]
        ii, jj = i + k.long(), j + ll.long()
        for a, b, w in ((0, 0, (1 - wx) * (1 - wy)), (0, 1, (1 - wx) * wy), (1, 0, wx * (1 - wy)), (1, 1, wx * wy)):
            add(2, ii + a, jj + b, c3 * w)

    # fields: planes with two ghost cells, row i at i + 2
    HALF = {"D": ((1, 0), (0, 1), (0, 0)), "B": ((0, 1), (1, 0), (1, 1))}

    def mesh(self):
        i = torch.arange(-2, self.n_r + 2, dtype=torch.float64, device=DEV)[:, None]
        j = torch.arange(-2, self.n_th + 2, dtype=torch.float64, device=DEV)[None, :]
        self.w = {(p, q): self.lower(i, p, j, q) for p in (0, 1) for q in (0, 1)}
        r = self.r0 + torch.exp(self.xi0 + (i + 0.5) * self.dxi)
        ra = r * r + self.a ** 2
        eta = 0.5 * self.dth
        th = eta + 2 * self.h0 * eta * (math.pi - 2 * eta) * (math.pi - eta) / math.pi ** 2
        self.cap = (self.dxi * (r - self.r0) * ra * torch.sqrt(1 + 2 * r / ra) * 2 * math.sin(0.5 * th) ** 2)[:, 0]

    def mirror(self, X, par, half):
        """Ghost columns by reflection in the axes."""
        n = self.n_th
        for k in (1, 2):
            X[:, 2 - k] = par * (X[:, 1 + k] if half else X[:, 2 + k])
            if n - half + k < n + 2:
                X[:, 2 + n - half + k] = par * X[:, 2 + n - k]
        return X

    def bounds(self, X, X0, kind):
        for k in range(3):
            h1, h2 = self.HALF[kind][k]
            X[k][:self.n_f + 3] = X[k][self.n_f + 3]
            if self.n_a:
                i = torch.arange(-2, self.n_r + 2, dtype=torch.float64, device=DEV)[:, None]
                lam = ((i + 0.5 * h1 - (self.n_r - self.n_a)) / self.n_a).clamp(0, 1) ** 3
                lam[:self.n_f + 3] = 0
                X[k] -= lam * (X[k] - X0[k])
            if (kind, k) in (("B", 1), ("D", 2)):
                X[k][:, 2] = X[k][:, 2 + self.n_th] = 0
            self.mirror(X[k], 1.0 if k == 0 else -1.0, h2)

    def aux(self, B, D):
        up = lambda X: torch.roll(X, -1, 0)  # noqa: E731
        dn = lambda X: torch.roll(X, 1, 0)  # noqa: E731
        n, h, t, m = self.w[0, 0], self.w[1, 0], self.w[0, 1], self.w[1, 1]
        fwd = lambda w, X, at: (w * X + up(w * X)) / (2 * at["sht"])  # noqa: E731
        bwd = lambda w, X, at: (w * X + dn(w * X)) / (2 * at["sht"])  # noqa: E731
        E = [h["al"] * (h["h11"] * D[0] + fwd(n["w13"], D[2], h)),
             t["al"] * t["h22"] * D[1] - bwd(m["wb"], B[2], t),
             n["al"] * (n["h33"] * D[2] + bwd(h["w13"], D[0], n)) + bwd(h["wb"], B[1], n)]
        H = [t["al"] * (t["h11"] * B[0] + bwd(m["w13"], B[2], t)),
             h["al"] * h["h22"] * B[1] + fwd(n["wb"], D[2], h),
             m["al"] * (m["h33"] * B[2] + fwd(t["w13"], B[0], m)) - fwd(t["wb"], D[1], m)]
        return E, H

    def faraday(self, B, E):
        n, t, dt = self.n_r, self.n_th, self.dt
        r, rr, c, cc = slice(2, n + 3), slice(2, n + 2), slice(2, t + 2), slice(3, t + 2)
        R, C = torch.roll, lambda X: torch.roll(X, -1, 1)
        w = self.w
        B[0][r, c] -= (dt * (C(E[2]) - E[2]) / w[0, 1]["sh"])[r, c]
        B[1][rr, cc] += (dt * (R(E[2], -1, 0) - E[2]) / w[1, 0]["sh"])[rr, cc]
        B[2][rr, c] -= (dt * ((R(E[1], -1, 0) - E[1]) - (C(E[0]) - E[0])) / w[1, 1]["sh"])[rr, c]

    def ampere(self, D, H, J):
        n, t, dt, pi = self.n_r, self.n_th, self.dt, math.pi
        r, rr, c, cc = slice(2, n + 3), slice(2, n + 2), slice(2, t + 2), slice(3, t + 2)
        R, w = torch.roll, self.w
        D[0][rr, cc] += (dt * (H[2] - R(H[2], 1, 1) - 4 * pi * J[0]) / w[1, 0]["sh"])[rr, cc]
        for col, h3 in ((2, H[2][:, 2]), (t + 2, -H[2][:, t + 1])):
            D[0][rr, col] += (dt * (h3 - 2 * pi * J[0][:, col]) / self.cap)[rr]
        D[1][r, c] += (dt * (-(H[2] - R(H[2], 1, 0)) - 4 * pi * J[1]) / w[0, 1]["sh"])[r, c]
        curl = (H[1] - R(H[1], 1, 0)) - (H[0] - R(H[0], 1, 1))
        D[2][r, cc] += (dt * (curl - 4 * pi * J[2]) / w[0, 0]["sh"])[r, cc]

    def smooth(self, X, par, half):
        for _ in range(self.n_f):
            S = self.mirror(X.clone(), par, half)
            t = torch.roll(S, 1, 1) + 2 * S + torch.roll(S, -1, 1)
            X = (torch.roll(t, 1, 0) + 2 * t + torch.roll(t, -1, 0)) / 16
            X[0], X[-1] = S[0], S[-1]
            c = slice(2, self.n_th + 3 - half)  # ghost columns take the source's reflection
            keep = X[:, c].clone()
            X = S
            X[:, c] = keep
        return X

    def start(self, F):
        """The advanced planes of a field set; in single precision with their low-order parts."""
        X = {k: F[p:p + 3].double() for k, p in grpic.PLANES.items() if k in ("D", "B", "D0", "B0", "J", "J0", "Dinit", "Binit")}
        if F.shape[0] > 33:
            X["D"], X["B"] = X["D"] + F[33:36].double(), X["B"] + F[36:39].double()
        self.mesh()
        return X

    def before(self, X):
        X["B0"] = 0.5 * (X["B0"] + X["B"])
        X["D0"] = 0.5 * (X["D0"] + X["D"])
        self.faraday(X["B0"], self.aux(X["B"], X["D0"])[0])
        self.bounds(X["B0"], X["Binit"], "B")

    def after(self, X):
        J = torch.stack([self.smooth(X["J"][k], 1.0 if k == 0 else -1.0, self.HALF["D"][k][1]) for k in range(3)])
        E, H = self.aux(X["B0"], X["D"])
        X["B0"] = X["B"].clone()
        self.faraday(X["B"], E)
        self.bounds(X["B"], X["Binit"], "B")
        self.ampere(X["D0"], H, 0.5 * (X["J0"] + J))
        self.bounds(X["D0"], X["Dinit"], "D")
        H = self.aux(X["B"], X["D0"])[1]
        X["D0"] = X["D"].clone()
        self.ampere(X["D"], H, J)
        self.bounds(X["D"], X["Dinit"], "D")
        X["J0"], X["J"] = J, torch.zeros_like(J)

    def planes(self, X):
        em = torch.cat([X["D"], X["B"], X["D0"], X["B0"]])
        return {"em": em} if _fp32(self.c) else {"em": em, "J0": X["J0"]}


def _wide(P):
    return {k: v.clone().long() if k in grpic.INT_FIELDS or k == "tag" else v.double() if v.dtype != torch.float64 else v.clone() for k, v in P.items()}


def _parts(P, most=1 << 24):
    """Views of consecutive slots, so that a large set's intermediates stay small."""
    return [{k: v[o:o + most] for k, v in P.items()} for o in range(0, P["tag"].numel(), most)]


def exact(case, seed):
    c = case
    cells, n = c["n_r"] * c["n_th"], 0 if c["kind"] == "fields" else _count(c)
    if c["kind"] == "inject" or cells > 5_000_000 or n * c.get("steps", 1) > 1_400_000_000:
        return None
    s = prepare(c, seed)
    x = _Exact(c, s["ctx"].dt)
    if c["kind"] == "frozen":
        F = _fields(c, s["ctx"], s["B0"])
        P = _wide(s["start"])
        for _ in range(c["steps"]):
            for part in _parts(P):
                x.push(part, F[0:3], F[9:12])
        final = torch.stack([P["i1"] + P["dx1"], P["i2"] + P["dx2"], P["u1"], P["u2"], P["u3"]], 1)
        return {"final": final, "g_u0": None, "g_B0": None} if c["grad"] else {"final": final}
    if c["kind"] == "diag":
        return _exact_diag(x, s)
    X = x.start(s["F0"])
    P = _wide(s["P0"]) if c["kind"] == "steps" else None
    for _ in range(c["steps"]):
        x.before(X)
        for part in _parts(P) if P is not None else ():
            x.deposit(X["J"], x.push(part, X["D"], X["B0"]))
        x.after(X)
    out = x.planes(X)
    if P is not None and not (c["sort"] or c["ranked"]):
        out.update(_particles(c, P))
    return out


def _exact_diag(x, s):
    """Energy and angular momentum at the time-centred position (the Wald potential included)."""
    P, a = _wide(s["P0"]), x.a
    x1 = 0.5 * (P["i1p"] + P["dx1p"] + P["i1"] + P["dx1"])
    x2 = 0.5 * (P["i2p"] + P["dx2p"] + P["i2"] + P["dx2"])
    r, _, sn, co, _ = x.at(x1, x2, True)
    Sg, ra = r * r + (a * co) ** 2, r * r + a * a
    A, z = ra * ra - a * a * (ra - 2 * r) * sn * sn, 2 * r / Sg
    A0 = 0.5 * s["B0"] * a * (z * (1 + co * co) - 2)
    A3 = 0.5 * s["B0"] * sn * sn * (A / Sg - 2 * a * a * z)
    al, b1, h11, h22, h33, h13 = x.upper(x1, x2)
    u1, u2, u3, t = P["u1"], P["u2"], P["u3"], P["tag"]
    q = torch.where(t == 1, 1.0, torch.where(t == 2, -1.0, 0.0)).double()
    g = torch.sqrt(1 + h11 * u1 * u1 + h22 * u2 * u2 + h33 * u3 * u3 + 2 * h13 * u1 * u3)
    return {"n_alive": None, "n_leaving": None, "n_empty": None, "n_nonfinite": None, "sum_E": None, "sum_L": None,
            "gauss_max": None, "gauss_scale": None, "E": al * g - b1 * u1 - q * A0, "L": u3 + q * A3, "gauss_res": None}
