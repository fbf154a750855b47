"""Performance cases of the two-belt pseudopotential lattice Boltzmann library.

Each case is one pass through the public entry points (Sim, Batch, Sim3, channel_loss) as a
program calls them: advance a lattice some steps and read its fields, take profiles of a Couette
cell, step a sweep of channels, monitor a run, or take a gradient.  listed() names the cases,
draw() gives more of the same ranges, prepare() makes a case's inputs and its simulation from a
seed, run() is one pass, work() its necessary bytes and operations, and exact() its outputs in
plain FP64 torch, written from eq. (LB) and eq. (FORCE) without this package.

Kinds of case (case["kind"]):
  run2d     Sim.step(steps), then moments()
  profiles  Couette cell: sample_profiles(samples, every), then profile_stats()
  monitor   reductions every step: step(steps), totals(), wall_stress(), stress_field(), checkpoint()
  sweep     Batch of channels of uneven size: step(steps) by graph, totals(), moments(i)
  adjoint   channel_loss(...) and its backward
  run3d     Sim3.step(steps), then moments() and totals()
"""

import math

import numpy as np
import torch

DEV = "cuda"
RICH, POOR = (1.2, 0.2), (0.2, 1.2)  # (rho_A, rho_B) of the droplets and of the continuous phase
G1, G2, GAB, RHO0 = (-9.0, -8.0), (8.1, 7.1), 0.587, 0.83  # emulsion couplings
FILM_G1, FILM_G2 = -20.4, 16.0  # one-component film couplings
ITEM = {"f64": 8, "f32": 4, "bf16dev": 2}


def listed():
    return [
        # the single-component relaxation run (64 x 64, FP64), fields read every 100 steps: the
        # smallest lattice, bound by latency
        dict(name="relax_64_f64", kind="run2d", lx=64, ly=64, ns=1, walls=False, storage="f64", start="noise", steps=100,
             graph=0, rounding="nearest"),
        # one point of the thin-film study (two bubbles of radius 64 pressed together): long FP64
        # runs of a small ragged lattice, replayed by graph
        dict(name="film_188x168_f64", kind="run2d", lx=188, ly=168, ns=1, walls=False, storage="f64", start="bubbles",
             steps=1000, graph=1000, rounding="nearest"),
        # the benchmark's emulsion, FP32 and FP64
        dict(name="emulsion_1024_f32", kind="run2d", lx=1024, ly=1024, ns=2, walls=False, storage="f32", start="drops",
             steps=50, graph=0, rounding="nearest"),
        dict(name="emulsion_1024_f64", kind="run2d", lx=1024, ly=1024, ns=2, walls=False, storage="f64", start="drops",
             steps=20, graph=0, rounding="nearest"),
        # the confined channel, FP32 and BF16 deviations with unbiased stores
        dict(name="channel_4096x512_f32", kind="run2d", lx=4096, ly=512, ns=2, walls=True, storage="f32", start="drops",
             steps=50, graph=0, rounding="nearest"),
        dict(name="channel_4096x512_bf16", kind="run2d", lx=4096, ly=512, ns=2, walls=True, storage="bf16dev",
             start="drops", steps=50, graph=0, rounding="stochastic"),
        # the planar Couette cell of the rheology runs: a profile every 20 steps and their statistics
        dict(name="couette_1040_f32", kind="profiles", lx=1040, ly=1040, ns=2, walls=True, storage="f32", samples=5, every=20),
        # a small channel watched closely: reductions every step, totals, stress and a checkpoint
        dict(name="monitor_320x200_f32", kind="monitor", lx=320, ly=200, ns=2, walls=True, storage="f32", steps=20),
        # a sweep of channels of uneven size and couplings stepped together
        dict(name="sweep_24_f32", kind="sweep", n=24, lx0=256, lx1=2048, ly0=64, ly1=512, ns=2, walls=True, storage="f32",
             steps=20, graph=20),
        # the gradient of wall stress and flow rate through the channel the adjoint is quoted on
        dict(name="adjoint_512x256", kind="adjoint", lx=512, ly=256, ns=2, walls=True, storage="f32", T=144, fp64_reverse=True),
        # three dimensions: the benchmark's emulsion in FP32, a ragged channel in FP64
        dict(name="emulsion3d_256_f32", kind="run3d", lx=256, ly=256, lz=256, ns=2, walls=False, storage="f32", steps=5),
        dict(name="channel3d_100x70x60_f64", kind="run3d", lx=100, ly=70, lz=60, ns=2, walls=True, storage="f64", steps=10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run2d", "run2d", "run2d", "profiles", "monitor", "sweep", "adjoint", "run3d"])
    storage = rng.choice(["f64", "f32", "f32", "bf16dev"])
    c = dict(kind=kind, ns=2, walls=rng.random() < 0.5, storage=storage)
    if kind == "run2d":
        c["lx"] = _log(rng, 48, 4096)
        c["ly"] = _log(rng, 48, min(1024, max(64, (1 << 21) // c["lx"])))
        c["ns"] = 1 if rng.random() < 0.35 else 2
        if c["ns"] == 1:
            c.update(start=rng.choice(["noise", "bubbles"]), walls=False, storage=rng.choice(["f64", "f64", "f32"]))
        else:
            c["start"] = "drops"
        sites = c["lx"] * c["ly"]
        c["steps"] = max(10, min(400, (1 << 25) // sites)) + rng.randrange(2)
        c["graph"] = rng.choice([0, 0, 10])
        c["rounding"] = rng.choice(["nearest", "stochastic"]) if c["storage"] == "bf16dev" else "nearest"
    elif kind == "profiles":
        c.update(walls=True, storage="f32", lx=_log(rng, 128, 1200), ly=_log(rng, 64, 1200), samples=rng.randrange(2, 7),
                 every=rng.randrange(5, 26))
    elif kind == "monitor":
        c.update(walls=True, storage=rng.choice(["f64", "f32"]), lx=_log(rng, 64, 1024), ly=_log(rng, 48, 512),
                 steps=rng.randrange(5, 31))
    elif kind == "sweep":
        c.update(walls=True, storage="f32", n=rng.randrange(3, 17), lx0=_log(rng, 64, 256), ly0=_log(rng, 32, 64), graph=10,
                 steps=20)
        c.update(lx1=_log(rng, 300, 1600), ly1=_log(rng, 72, 400))
    elif kind == "adjoint":
        c.update(walls=True, storage=rng.choice(["f32", "f64"]), lx=_log(rng, 64, 512), ly=_log(rng, 32, 256),
                 T=rng.randrange(30, 145), fp64_reverse=rng.random() < 0.5)
    else:
        c.update(storage=rng.choice(["f64", "f32"]), lx=_log(rng, 32, 200), ly=_log(rng, 32, 160), lz=_log(rng, 24, 160),
                 steps=rng.randrange(4, 11))
    return c


# ---------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------

def _drops(shape, seed, walls):
    """Packed droplets: density [2, *shape] (host FP64) of a jittered lattice of centres about 28
    sites apart (20 in three dimensions); a site is A-rich where the second nearest centre is at
    least two sites further off than the nearest, so thin B films separate the droplets."""
    g = np.random.Generator(np.random.PCG64(seed))
    size = 28.0 if len(shape) == 2 else 20.0
    cells = [max(3, int(round(n / size))) for n in shape]
    centres = g.uniform(0.15, 0.85, (*cells, len(shape)))  # of each cell's extent
    centres = torch.as_tensor(centres, dtype=torch.float32, device=DEV)
    axes = [torch.arange(n, device=DEV, dtype=torch.float32) + 0.5 for n in shape]
    width = [n / k for n, k in zip(shape, cells)]
    home = [torch.clamp((a / w).floor().long(), max=k - 1) for a, w, k in zip(axes, width, cells)]
    d1 = torch.full(shape, 1e9, device=DEV)
    d2 = torch.full(shape, 1e9, device=DEV)
    for o in np.ndindex(*([3] * len(shape))):
        at = [h + (s - 1) for h, s in zip(home, o)]
        idx = torch.meshgrid(*[a % k for a, k in zip(at, cells)], indexing="ij")
        d = torch.zeros(shape, device=DEV)
        for k in range(len(shape)):
            view = [1] * len(shape)
            view[k] = shape[k]
            d += (axes[k].view(view) - (at[k].float().view(view) + centres[..., k][idx]) * width[k]) ** 2
        d = d.sqrt()
        d2 = torch.minimum(d2, torch.maximum(d1, d))
        d1 = torch.minimum(d1, d)
    rich = (d2 - d1) >= 2.0
    if walls:  # a B film along both walls (rows are the second axis from the right)
        rich = rich.clone()
        rich[..., 0, :] = False
        rich[..., -1, :] = False
    rho = torch.stack([torch.where(rich, RICH[s], POOR[s]) for s in range(2)]).double()
    return rho.cpu().numpy()


def _bubbles(lx, ly, seed):
    """Two gas bubbles facing each other across a liquid film, with a seeded position, size and gap."""
    g = np.random.Generator(np.random.PCG64(seed))
    radius = max(4.0, 0.5 * (min(lx, ly) - 40) * g.uniform(0.9, 1.0))
    gap = g.uniform(5.0, 7.0)
    y, x = np.mgrid[0:ly, 0:lx] + 0.5
    xl, xr, cy = lx / 2.0 - gap / 2.0, lx / 2.0 + gap / 2.0, ly / 2.0
    dl = np.maximum(np.hypot(x - xl, y - cy) - radius, x - xl)
    dr = np.maximum(np.hypot(x - xr, y - cy) - radius, xr - x)
    return 0.28 + 1.11 * 0.5 * (1.0 + np.tanh(np.minimum(dl, dr) / 1.5))


def _noise(shape, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    return 1.0 + 0.01 * g.uniform(-1.0, 1.0, shape)


def _params(c, seed):
    """Density and parameters of a single-lattice case, as Sim's keyword arguments."""
    if c["ns"] == 1:
        lx, ly = c["lx"], c["ly"]
        rho = _bubbles(lx, ly, seed) if c["start"] == "bubbles" else _noise((ly, lx), seed)
        return rho[None], dict(n_species=1, walls=False, g1=(FILM_G1, 0.0), g2=(FILM_G2, 0.0), tau=(1.0, 1.0), psi0=1.0,
                               rho0=1.0)
    rho = _drops((c["ly"], c["lx"]), seed, c["walls"])
    kw = dict(n_species=2, walls=c["walls"], g1=G1, g2=G2, gab=GAB, tau=(1.0, 1.0), psi0=1.0, rho0=RHO0)
    if c["walls"]:
        kw["rho_wall"] = POOR
        if c["kind"] == "profiles":
            kw["u_wall"] = (-0.01, 0.01)
        else:
            kw["body"] = (1e-6, 0.0)
    if c["kind"] == "adjoint":
        kw.update(g1=(-9.0, -9.0), g2=(8.1, 8.1))
    return rho, kw


def _sweep(c, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    sizes = np.random.Generator(np.random.PCG64(c["n"]))  # the same sizes for every seed
    out = []
    for i in range(c["n"]):
        lx, ly = int(sizes.integers(c["lx0"], c["lx1"] + 1)), int(sizes.integers(c["ly0"], c["ly1"] + 1))
        e = g.uniform(-1.0, 1.0, 6)
        out.append(dict(lx=lx, ly=ly, rho_init=_drops((ly, lx), seed * 1000 + i, True),
                        g1=tuple(G1[s] * (1 + 0.05 * e[s]) for s in range(2)),
                        g2=tuple(G2[s] * (1 + 0.05 * e[2 + s]) for s in range(2)), gab=GAB * (1 + 0.1 * e[4]),
                        body=(1e-6 * (1.25 + 0.75 * e[5]), 0.0), rho_wall=POOR, tau=(1.0, 1.0), psi0=1.0, rho0=RHO0))
    return out


def _populations(rho):
    """Canonical rest populations W_l rho, [ns, 9, ly, lx] on the device."""
    w = torch.tensor([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4, dtype=torch.float64, device=DEV)
    return (w[None, :, None, None] * torch.as_tensor(rho, device=DEV)[:, None]).contiguous()


def prepare(case, seed):
    from paper_1402_6019_amd import Batch, Sim, Sim3
    c = case
    if c["kind"] == "sweep":
        b = Batch(_sweep(c, seed), n_species=2, walls=True, storage=c["storage"])
        b.set_graph(c["graph"])
        return dict(case=c, batch=b)
    if c["kind"] == "run3d":
        rho = _drops((c["lz"], c["ly"], c["lx"]), seed, c["walls"])
        kw = dict(body=(1e-6, 0.0, 0.0), rho_wall=POOR) if c["walls"] else {}
        return dict(case=c, sim=Sim3(c["lx"], c["ly"], c["lz"], rho, n_species=2, walls=c["walls"], storage=c["storage"],
                                     g1=G1, g2=G2, gab=GAB, tau=(1.0, 1.0), psi0=1.0, rho0=RHO0, **kw))
    rho, kw = _params(c, seed)
    sim = Sim(c["lx"], c["ly"], rho, storage=c["storage"], **kw)
    state = dict(case=c, sim=sim)
    if c["kind"] == "run2d":
        if c["rounding"] != "nearest":
            sim.set_rounding(c["rounding"])
        if c["graph"]:
            sim.set_graph(c["graph"])
    elif c["kind"] == "monitor":
        sim.set_reduce_every(1)
    elif c["kind"] == "adjoint":
        state["f0"] = _populations(rho)
        state["theta"] = torch.tensor([*kw["g1"], *kw["g2"], kw["gab"], kw["body"][0]], dtype=torch.float64)
    return state


def run(state):
    c, kind = state["case"], state["case"]["kind"]
    out = torch.float64 if c["storage"] == "f64" else torch.float32
    if kind == "sweep":
        b = state["batch"]
        b.step(c["steps"])
        return dict(totals=b.totals(), fields=[b.moments(i, dtype=out) for i in range(c["n"])])
    sim = state["sim"]
    if kind == "run2d":
        sim.step(c["steps"])
        return sim.moments(dtype=out)
    if kind == "run3d":
        sim.step(c["steps"])
        return dict(fields=sim.moments(dtype=out), totals=sim.totals())
    if kind == "profiles":
        samples = sim.sample_profiles(c["samples"], c["every"])
        return dict(samples=samples, stats=sim.profile_stats(samples))
    if kind == "monitor":
        sim.step(c["steps"])
        return dict(totals=sim.totals(), wall=sim.wall_stress(reset=True), stress=sim.stress_field(dtype=out),
                    f=sim.checkpoint())
    from paper_1402_6019_amd.adjoint import channel_loss
    theta = state["theta"].clone().requires_grad_(True)
    loss = channel_loss(theta, sim, state["f0"], c["T"], (1.0, 1.0), fp64_reverse=c["fp64_reverse"])
    loss.backward()
    return dict(loss=loss.detach(), grad=theta.grad, fields=sim.moments(dtype=out))


def work(case):
    """Every step reads and writes each population once (the bytes of a lattice update that the
    library reports), outputs are written once; a reverse step reads and writes the adjoint
    populations and reads the state's moments."""
    c = case
    item, ns = ITEM[c["storage"]], c["ns"]
    out = 8 if c["storage"] == "f64" else 4
    site2, flops2 = 2 * 9 * ns * item, 225.0 * ns
    if c["kind"] == "sweep":
        sizes = np.random.Generator(np.random.PCG64(c["n"]))
        n = sum(int(sizes.integers(c["lx0"], c["lx1"] + 1)) * int(sizes.integers(c["ly0"], c["ly1"] + 1))
                for _ in range(c["n"]))
        return {"bytes": float(n * (c["steps"] * site2 + 9 * ns * item * 2 + (ns + 2) * out)),
                "flops": n * c["steps"] * flops2}
    n = c["lx"] * c["ly"]
    if c["kind"] == "run3d":
        n *= c["lz"]
        return {"bytes": float(n * (c["steps"] * 2 * 19 * ns * item + 2 * 19 * ns * item + (ns + 3) * out)),
                "flops": n * c["steps"] * 600.0 * ns}
    if c["kind"] == "run2d":
        return {"bytes": float(n * (c["steps"] * site2 + 9 * ns * item + (ns + 2) * out)), "flops": n * c["steps"] * flops2}
    if c["kind"] == "profiles":
        return {"bytes": float(n * c["samples"] * (c["every"] * site2 + 9 * ns * item)),
                "flops": n * c["samples"] * (c["every"] + 1) * flops2}
    if c["kind"] == "monitor":
        return {"bytes": float(n * (c["steps"] * site2 + 3 * 9 * ns * item + 3 * out + 9 * ns * 8)),
                "flops": n * (c["steps"] + 2) * flops2}
    r = 8 if c["fp64_reverse"] or c["storage"] == "f64" else 4
    return {"bytes": float(n * (c["T"] * (site2 + 2 * 4 * ns * r + 2 * 9 * ns * r) + 9 * ns * 8)),
            "flops": n * c["T"] * 3.5 * flops2}


# ---------------------------------------------------------------------------------------
# The same in plain FP64 torch
# ---------------------------------------------------------------------------------------

C9 = ((0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1))
W9 = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4
OPP9 = (0, 3, 4, 1, 2, 7, 8, 5, 6)
SHELL2 = {1: 0, 2: 1, 4: 2, 5: 3, 8: 4}
WA2 = (4 / 45, 1 / 30, 1 / 360, 0.0, 0.0)
PA2 = (4 / 63, 4 / 135, 1 / 180, 2 / 945, 1 / 15120)
T2 = {1: 1 / 9, 2: 1 / 36}


class _Plane:
    """Two-dimensional lattice in FP64: f [ns, 9, ly, lx] holds pre-collision populations."""

    def __init__(self, rho, kw):
        self.ns, self.ly, self.lx = rho.shape
        self.walls = kw["walls"]
        z = (0.0, 0.0)
        self.g1, self.g2, self.gab = kw["g1"], kw["g2"], kw.get("gab", 0.0)
        self.body, self.rw, self.uw = kw.get("body", z), kw.get("rho_wall", z), kw.get("u_wall", z)
        self.tau, self.psi0, self.rho0 = kw["tau"], kw["psi0"], kw["rho0"]
        self.f = _populations(rho)

    def psi(self, rho):
        return self.psi0 * (1.0 - torch.exp(-rho / self.rho0))

    def padded(self, v, wall):
        """v with two more sites on every side: periodic in x, periodic or wall ghosts in y."""
        v = torch.cat([v[:, -2:], v, v[:, :2]], 1)
        if self.walls:
            ghost = torch.full((2, v.shape[1]), float(wall), dtype=v.dtype, device=v.device)
            return torch.cat([ghost, v, ghost], 0)
        return torch.cat([v[-2:], v, v[:2]], 0)

    def at(self, p, cx, cy):
        return p[2 + cy:2 + cy + self.ly, 2 + cx:2 + cx + self.lx]

    def fields(self):
        """rho, j, F and the neighbourhoods of psi and rho."""
        f, ns = self.f, self.ns
        rho = [f[s].sum(0) for s in range(ns)]
        jx = [sum(C9[l][0] * f[s, l] for l in range(9) if C9[l][0]) for s in range(ns)]
        jy = [sum(C9[l][1] * f[s, l] for l in range(9) if C9[l][1]) for s in range(ns)]
        psi = [self.psi(r) for r in rho]
        pp = [self.padded(psi[s], self.psi0 * (1.0 - math.exp(-self.rw[s] / self.rho0))) for s in range(ns)]
        rp = [self.padded(rho[s], self.rw[s]) for s in range(ns)]
        fx, fy = [], []
        for s in range(ns):
            ax, ay = torch.zeros_like(rho[s]), torch.zeros_like(rho[s])
            for cx in range(-2, 3):
                for cy in range(-2, 3):
                    q = SHELL2.get(cx * cx + cy * cy)
                    if q is not None:
                        k = self.g1[s] * WA2[q] + self.g2[s] * PA2[q]
                        v = k * self.at(pp[s], cx, cy)
                        ax, ay = ax + cx * v, ay + cy * v
            x, y = -psi[s] * ax, -psi[s] * ay
            if ns == 2:
                o = 1 - s
                bx, by = torch.zeros_like(x), torch.zeros_like(x)
                for cx, cy in C9[1:]:
                    v = T2[cx * cx + cy * cy] * self.at(rp[o], cx, cy)
                    bx, by = bx + cx * v, by + cy * v
                x, y = x - self.gab * rho[s] * bx, y - self.gab * rho[s] * by
            fx.append(x + rho[s] * self.body[0])
            fy.append(y + rho[s] * self.body[1])
        return rho, psi, jx, jy, fx, fy, pp, rp

    def velocity(self, fl):
        rho, _, jx, jy, fx, fy = fl[:6]
        m = sum(rho)
        return [sum(j[s] + 0.5 * F[s] for s in range(self.ns)) / m for j, F in ((jx, fx), (jy, fy))]

    def collide(self, fl):
        rho, _, jx, jy, fx, fy = fl[:6]
        den = sum(rho[s] / self.tau[s] for s in range(self.ns))
        upx = sum(jx[s] / self.tau[s] for s in range(self.ns)) / den
        upy = sum(jy[s] / self.tau[s] for s in range(self.ns)) / den
        out = []
        for s in range(self.ns):
            ux, uy = upx + self.tau[s] * fx[s] / rho[s], upy + self.tau[s] * fy[s] / rho[s]
            uu = ux * ux + uy * uy
            eq = []
            for (cx, cy), w in zip(C9, W9):
                cu = cx * ux + cy * uy
                eq.append(w * rho[s] * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu))
            out.append(self.f[s] + (torch.stack(eq) - self.f[s]) / self.tau[s])
        return torch.stack(out)

    def stream(self, g):
        new = []
        for s in range(self.ns):
            row = []
            for l, (cx, cy) in enumerate(C9):
                v = torch.roll(g[s, l], (cy, cx), (0, 1))
                if self.walls and cy:
                    # W_l rho_w 6 (c_l . U): the momentum a moving wall hands the reflected population
                    y, wall = (0, 0) if cy > 0 else (self.ly - 1, 1)
                    back = g[s, OPP9[l], y] + 6.0 * W9[l] * self.rw[s] * cx * self.uw[wall]
                    v = torch.cat([back[None], v[1:]]) if cy > 0 else torch.cat([v[:-1], back[None]])
                row.append(v)
            new.append(torch.stack(row))
        return torch.stack(new)

    def wall_force(self, g):
        bot = top = 0.0
        for s in range(self.ns):
            bot = bot + 2.0 * (g[s, 8, 0] - g[s, 7, 0]).sum() / self.lx - self.rw[s] * self.uw[0] / 3.0
            top = top + 2.0 * (g[s, 5, -1] - g[s, 6, -1]).sum() / self.lx - self.rw[s] * self.uw[1] / 3.0
        return bot, top

    def step(self):
        g = self.collide(self.fields())
        self.f = self.stream(g)
        return g

    def moments(self):
        fl = self.fields()
        return torch.stack(fl[0]), torch.stack(self.velocity(fl))

    def totals(self):
        fl = self.fields()
        m = [float(r.sum()) for r in fl[0]] + [0.0] * (2 - self.ns)
        p = (float(sum(j.sum() for j in fl[2])), float(sum(j.sum() for j in fl[3])))
        return (m[0], m[1]), p, float(self.velocity(fl)[0].sum() / self.lx)

    def profile(self):
        fl = self.fields()
        rho, psi, _, _, _, _, pp, rp = fl
        g = self.collide(fl)
        kup = sum((g[s, 5] - g[s, 6]).sum(1) for s in range(self.ns))
        kdn = sum((g[s, 8] - g[s, 7]).sum(1) for s in range(self.ns))
        i1 = i2 = 0.0  # x-force on a row from partners at c_y = 1 and from those at c_y = 2
        for s in range(self.ns):
            for cx in (-2, -1, 1, 2):
                for cy in (1, 2):
                    q = SHELL2[cx * cx + cy * cy]
                    k = self.g1[s] * WA2[q] + self.g2[s] * PA2[q]
                    v = -(k * cx * psi[s] * self.at(pp[s], cx, cy)).sum(1)
                    i1, i2 = (i1 + v, i2) if cy == 1 else (i1, i2 + v)
            if self.ns == 2:
                for cx in (-1, 1):
                    i1 = i1 - (self.gab / 36.0 * cx * rho[s] * self.at(rp[1 - s], cx, 1)).sum(1)
        i1 = i1 + i2
        up = lambda v, k: torch.roll(v, k)  # noqa: E731
        i2s = up(i2, 2)
        if self.walls:
            i2s = i2s.clone()
            i2s[:2] = 0.0
        sig = (up(i1, 1) + i2s - up(kup, 1) + kdn) / self.lx
        if self.walls:
            wb, wt = self.wall_force(g)
            sig = torch.cat([wb[None], sig[1:], -wt[None]])
        else:
            sig = torch.cat([sig, sig[:1]])
        ra, rb = rho[0].mean(1), rho[1].mean(1)
        return torch.cat([self.velocity(fl)[0].mean(1), sig, ra, rb])

    def stress(self):
        """Pressure tensor of Appendix A, shell by shell."""
        rho, psi, _, _, fx, fy, pp, rp = self.fields()
        sig = [torch.zeros_like(rho[0]) for _ in range(3)]

        def add(k, v, cx, cy):
            for i, w in enumerate((cx * cx, cx * cy, cy * cy)):
                if w:
                    sig[i].add_(k * w * v)

        for s in range(self.ns):
            n = lambda cx, cy: self.at(pp[s], cx, cy)  # noqa: B023, E731
            for cx in range(-2, 3):
                for cy in range(-2, 3):
                    q = SHELL2.get(cx * cx + cy * cy)
                    if q is None:
                        continue
                    k = self.g1[s] * WA2[q] + self.g2[s] * PA2[q]
                    if q < 2:
                        add(0.5 * k, psi[s] * n(cx, cy), cx, cy)
                    elif q in (2, 4):
                        hx, hy = cx // 2, cy // 2
                        add(0.25 * k, psi[s] * n(cx, cy) + n(-hx, -hy) * n(hx, hy), cx, cy)
                    else:  # (2, 1): the pair at its ends, and the two pairs between whose sites it lies
                        ax, ay = (int(math.copysign(1, cx)), int(math.copysign(1, cy)))
                        if abs(cx) == 2:
                            between = n(ax, ay) * n(-ax, 0) + n(ax, 0) * n(-ax, -ay)
                        else:
                            between = n(ax, ay) * n(0, -ay) + n(0, ay) * n(-ax, -ay)
                        add(0.25 * k, psi[s] * n(cx, cy) + 0.5 * between, cx, cy)
            c = (self.tau[s] - 0.5) ** 2 / rho[s]
            sig[0] += rho[s] / 3.0 + c * fx[s] * fx[s]
            sig[1] += c * fx[s] * fy[s]
            sig[2] += rho[s] / 3.0 + c * fy[s] * fy[s]
        if self.ns == 2:
            for s in range(2):
                for cx, cy in C9[1:]:
                    add(0.5 * self.gab * T2[cx * cx + cy * cy], rho[s] * self.at(rp[1 - s], cx, cy), cx, cy)
        return torch.stack(sig)


C19 = ((0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0), (1, -1, 0),
       (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1))
W19 = (1 / 3,) + (1 / 18,) * 6 + (1 / 36,) * 12


class _Box:
    """Three-dimensional lattice in FP64, species by species to bound the memory; the shell weights
    are the library's documented defaults."""

    def __init__(self, rho, walls):
        from paper_1402_6019_amd import _binding as B
        import ctypes
        d = B.Lb3Couplings()
        B.load().lb3_default_couplings(ctypes.byref(d))
        self.w, self.p = list(d.w), list(d.p)  # shells |c|^2 = 1, 2, 3, 4, 5, 6, 8 (inputs of the model)
        self.ns, self.lz, self.ly, self.lx = rho.shape
        self.walls = walls
        self.rw = POOR if walls else (0.0, 0.0)
        self.body = 1e-6 if walls else 0.0
        r = torch.as_tensor(rho, device=DEV)
        self.f = [[W19[l] * r[s] for l in range(19)] for s in range(2)]

    def pad(self, v, wall):
        v = torch.cat([v[..., -2:], v, v[..., :2]], 2)
        if self.walls:
            g = torch.full((v.shape[0], 2, v.shape[2]), float(wall), dtype=v.dtype, device=v.device)
            v = torch.cat([g, v, g], 1)
        else:
            v = torch.cat([v[:, -2:], v, v[:, :2]], 1)
        return torch.cat([v[-2:], v, v[:2]], 0)

    def at(self, p, c):
        return p[2 + c[2]:2 + c[2] + self.lz, 2 + c[1]:2 + c[1] + self.ly, 2 + c[0]:2 + c[0] + self.lx]

    def fields(self):
        rho = [sum(f[1:], f[0].clone()) for f in self.f]
        j = [[sum((f[l] if C19[l][k] > 0 else -f[l]) for l in range(19) if C19[l][k]) for k in range(3)] for f in self.f]
        shell = {1: 0, 2: 1, 3: 2, 4: 3, 5: 4, 6: 5, 8: 6}
        rp = [self.pad(rho[s], self.rw[s]) for s in range(2)]
        F = []
        for s in range(2):
            psi = 1.0 - torch.exp(-rho[s] / RHO0)
            pp = self.pad(psi, 1.0 - math.exp(-self.rw[s] / RHO0))
            a = [torch.zeros_like(psi) for _ in range(3)]
            for cz in range(-2, 3):
                for cy in range(-2, 3):
                    for cx in range(-2, 3):
                        q = shell.get(cx * cx + cy * cy + cz * cz)
                        if q is None:
                            continue
                        v = self.at(pp, (cx, cy, cz))
                        k = G1[s] * self.w[q] + G2[s] * self.p[q]
                        for i, e in enumerate((cx, cy, cz)):
                            if e:
                                a[i].add_(v, alpha=k * e)
            a = [-psi * v for v in a]
            for l in range(1, 19):
                v = rho[s] * self.at(rp[1 - s], C19[l])
                t = (1 / 18) if l < 7 else (1 / 36)
                for i, e in enumerate(C19[l]):
                    if e:
                        a[i].add_(v, alpha=-GAB * t * e)
            a[0].add_(rho[s], alpha=self.body)
            F.append(a)
        return rho, j, F

    def step(self):
        rho, j, F = self.fields()
        m = rho[0] + rho[1]
        up = [(j[0][k] + j[1][k]) / m for k in range(3)]
        for s in range(2):
            u = [up[k] + F[s][k] / rho[s] for k in range(3)]
            uu = sum(v * v for v in u)
            g = []
            for l in range(19):  # tau = 1: the post-collision populations are the equilibrium
                cu = sum((u[k] if C19[l][k] > 0 else -u[k]) for k in range(3) if C19[l][k]) if l else torch.zeros_like(uu)
                g.append(W19[l] * rho[s] * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu))
            for l in range(19):
                cx, cy, cz = C19[l]
                v = torch.roll(g[l], (cz, cy, cx), (0, 1, 2))
                if self.walls and cy:
                    y = 0 if cy > 0 else self.ly - 1
                    v[:, y] = g[l + 1 if l % 2 else l - 1][:, y]
                self.f[s][l] = v

    def result(self):
        rho, j, F = self.fields()
        m = rho[0] + rho[1]
        u = torch.stack([(j[0][k] + j[1][k] + 0.5 * (F[0][k] + F[1][k])) / m for k in range(3)])
        mom = [float(j[0][k].sum() + j[1][k].sum()) for k in range(3)]
        return torch.stack(rho), u, [float(r.sum()) for r in rho], mom, float(u[0].sum())


def _gradient(c, rho, kw):
    p = _Plane(rho, kw)
    th = [torch.tensor(v, dtype=torch.float64, device=DEV, requires_grad=True)
          for v in (*kw["g1"], *kw["g2"], kw["gab"], kw["body"][0])]
    p.g1, p.g2, p.gab, p.body = (th[0], th[1]), (th[2], th[3]), th[4], (th[5], 0.0)

    def one(f, *_):
        p.f = f
        fl = p.fields()
        g = p.collide(fl)
        wb, wt = p.wall_force(g)
        return p.stream(g), 0.5 * (wb + wt) + p.velocity(fl)[0].sum() / p.lx

    loss, f = 0.0, p.f
    for _ in range(c["T"]):
        f, v = torch.utils.checkpoint.checkpoint(one, f, *th, use_reentrant=False)
        loss = loss + v / c["T"]
    loss.backward()
    p.f = f.detach()
    p.g1, p.g2, p.gab, p.body = kw["g1"], kw["g2"], kw["gab"], kw["body"]
    return dict(loss=loss.detach().cpu(), grad=torch.stack([t.grad for t in th]).cpu(), fields=p.moments())


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "run3d":
        b = _Box(_drops((c["lz"], c["ly"], c["lx"]), seed, c["walls"]), c["walls"])
        for _ in range(c["steps"]):
            b.step()
        rho, u, mass, mom, ux = b.result()
        # the total momentum and flow of a lattice nearly at rest are what rounding leaves of sums that cancel
        return dict(fields=(rho, u), totals=(mass, None, None))
    if kind == "sweep":
        tot, fields = [], []
        for inst in _sweep(c, seed):
            kw = {k: v for k, v in inst.items() if k not in ("lx", "ly", "rho_init")}
            p = _Plane(inst["rho_init"], dict(kw, walls=True))
            for _ in range(c["steps"]):
                p.step()
            m, mo, q = p.totals()
            tot.append([*m, *mo, q])
            fields.append(p.moments())
        return dict(totals=np.array(tot), fields=fields)
    rho, kw = _params(c, seed)
    if kind == "adjoint":
        return _gradient(c, rho, kw)
    p = _Plane(rho, kw)
    if kind == "run2d":
        for _ in range(c["steps"]):
            p.step()
        return p.moments()
    if kind == "monitor":
        wall = []
        for _ in range(c["steps"]):
            wall.append(p.wall_force(p.step()))
        return dict(totals=(p.totals()[0], None, None), wall=tuple(float(sum(w[k] for w in wall)) / len(wall) for k in range(2)),
                    stress=p.stress(), f=p.f)
    samples = []
    for _ in range(c["samples"]):
        for _ in range(c["every"]):
            p.step()
        samples.append(p.profile())
    x, ly = torch.stack(samples), c["ly"]
    mean = x.mean(0)
    # the fluidity divides by stresses that pass through zero and the correlator by their variance
    # over a few samples: no value to hold FP32 runs to
    return dict(samples=x, stats=dict(u=mean[:ly], sigma=mean[ly:2 * ly + 1], fluidity=None, corr=None,
                                      rho_a=mean[2 * ly + 1:3 * ly + 1], rho_b=mean[3 * ly + 1:]))
