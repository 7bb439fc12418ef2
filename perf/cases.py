"""The calls whose time counts, for measuring one version of the library
against another: inputs and handles as a simulation program keeps them, one
pass through the public entry points, the work a pass cannot do without, and
the same results from plain torch in 64 bits.

A pass of a stepping case is one `Simulation.step(n)` and the read-out a
program makes after it (the fields it plots, or the updated state it keeps);
the state moves on from pass to pass.  The seed draws where the droplets sit,
where the carrier flow points and a small velocity noise.
"""
import math

import numpy as np
import torch

import paper_2309_07801_amd as pkg

STORAGE = {"fp32": pkg.FP32, "fp32_pairs": pkg.FP32_PAIRS, "fp32_exact": pkg.FP32_EXACT,
           "fp16": pkg.FP16_SHIFT, "bf16": pkg.BF16_SHIFT, "fp16c": pkg.FP16_CSHIFT,
           "bf16c": pkg.BF16_CSHIFT}
FIELDS = ("rho_r", "rho_b", "phi", "p", "ux", "uy", "uz")

# What a case leaves unsaid.
#   flow: droplet (one droplet carried obliquely through a periodic box),
#     field (a jittered grid of droplets, D2Q9), collision (two droplets head
#     on between walls in y and z), layer (heavy over light, walls in z)
#   sigma: interfacial tension over the light phase's density
#   schedule: default (what the handle starts with), tuned (what the
#     autotuner picks), compact (tuned, then schedule 2)
#   read: state (the stored populations), fields (densities and velocity),
#     monitor (the diagnostics and seven fields; no step)
DEFAULTS = dict(lattice="d3q27", flow="droplet", boxes=1, gamma=10.0, tau=0.625, sigma=0.05,
                radius=0.125, speed=0.05, storage="fp32", schedule="compact", resident=False,
                inplace=False, model=3, rate=1.0, steps=10, read="fields")


def _full(case):
    return dict(DEFAULTS, **case)


def listed():
    return [
        # the smallest call: a 32^3 static-droplet box, a few steps at a time
        # (launches and latency)
        dict(name="droplet 32 cube", nx=32, ny=32, nz=32, gamma=1.0, tau=1.0, sigma=0.01,
             radius=0.25, speed=0.02, schedule="tuned", steps=10, read="state"),
        # the main workload: a 256^3 translating droplet, density ratio 10,
        # compact state kept between calls, fields read after every 20 steps
        dict(name="droplet 256 cube", nx=256, ny=256, nz=256, resident=True, steps=20),
        # a handle used as it comes: default schedule, no autotuning, a box
        # that no tile divides, a few steps per call
        dict(name="droplet default schedule", nx=200, ny=144, nz=177, schedule="default", steps=4,
             read="state"),
        # 16-bit storage in the compact schedule, odd extents
        dict(name="droplet fp16", nx=190, ny=131, nz=150, storage="fp16", steps=10),
        # 16-bit storage in the population schedule (rounded at every step)
        dict(name="droplet bf16c population", nx=128, ny=112, nz=96, storage="bf16c",
             schedule="tuned", steps=4),
        # per-colour mass exact to FP64
        dict(name="droplet mass exact", nx=160, ny=160, nz=160, storage="fp32_exact", steps=10),
        # a sweep of independent boxes of 24 to 128 nodes an edge in one handle
        dict(name="batch of 24 boxes", boxes=24, lmin=24, lmax=128, box_seed=4, radius=0.25,
             sigma=0.03, storage="fp32_pairs", resident=True, steps=10, read="state"),
        # the walled head-on collision at half its published size
        dict(name="collision", flow="collision", nx=384, ny=192, nz=192, tau=0.55, radius=0.125,
             resident=True, steps=10, read="state"),
        # Rayleigh-Taylor with the standard equilibrium (model comparison)
        dict(name="layer model A", flow="layer", nx=96, ny=96, nz=384, gamma=3.0, sigma=0.0,
             tau=0.52, model=0, steps=10, read="state"),
        # relaxation rates above second order other than one
        dict(name="droplet general rates", nx=97, ny=80, nz=113, rate=1.2, schedule="tuned",
             steps=4, read="state"),
        # the two-dimensional model on a field of droplets
        dict(name="d2q9 field", lattice="d2q9", flow="field", nx=2048, ny=2048, nz=1,
             schedule="tuned", steps=10, read="state"),
        # what a run reads between its steps: diagnostics and seven fields
        dict(name="monitor", nx=192, ny=192, nz=192, steps=0, read="monitor"),
    ]


def draw(rng):
    def edge(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("compact", "compact", "compact", "population", "population", "batch",
                       "collision", "layer", "rates", "d2q9", "d2q9", "monitor"))
    c = {"gamma": rng.choice((1.0, 2.0, 3.0, 10.0))}
    if kind == "d2q9":
        c.update(lattice="d2q9", flow="field", nx=edge(64, 4096), ny=edge(64, 4096), nz=1,
                 schedule=rng.choice(("default", "tuned")),
                 storage=rng.choice(("fp32", "fp16", "bf16", "fp32_exact")))
        c["steps"] = rng.choice((1, 4, 10))
        c["read"] = "state" if c["storage"] == "fp32" else "fields"
        return c
    if kind == "batch":
        lo = rng.randint(20, 48)
        c.update(boxes=rng.randint(3, 24), lmin=lo, lmax=rng.randint(lo + 8, 128),
                 box_seed=rng.randint(0, 10 ** 6), radius=0.25, sigma=0.03,
                 storage=rng.choice(("fp32_pairs", "fp32")),
                 schedule=rng.choice(("compact", "tuned")), steps=rng.choice((2, 5, 10)),
                 read="state")
        c["resident"] = c["schedule"] == "compact"
        return c
    c.update(nx=edge(24, 288), ny=edge(24, 256), nz=edge(24, 256))
    if kind == "collision":
        c.update(flow="collision", nx=2 * edge(40, 180), ny=edge(48, 200), nz=edge(48, 200),
                 tau=0.55, resident=rng.random() < 0.5, steps=rng.choice((4, 10)), read="state",
                 storage=rng.choice(("fp32", "fp32_pairs")))
    elif kind == "layer":
        c.update(flow="layer", gamma=3.0, sigma=0.0, tau=0.52, model=rng.choice((0, 3)),
                 steps=rng.choice((4, 10)), read="state")
    elif kind == "rates":
        c.update(rate=rng.choice((0.9, 1.1, 1.2)), schedule=rng.choice(("default", "tuned")),
                 steps=rng.choice((2, 4)), read="state")
    elif kind == "monitor":
        c.update(steps=0, read="monitor", storage=rng.choice(("fp32", "fp16c")),
                 schedule="default")
    elif kind == "population":
        c.update(schedule=rng.choice(("default", "tuned")), steps=rng.choice((1, 4, 8)),
                 storage=rng.choice(("fp32", "fp16", "bf16c", "fp32_exact")),
                 inplace=rng.random() < 0.3)
        c["read"] = "state" if c["storage"] == "fp32" else "fields"
    else:
        c.update(storage=rng.choice(("fp32", "fp32", "fp16", "bf16c", "fp32_exact")),
                 steps=rng.choice((3, 10, 20)))
        c["resident"] = c["storage"] == "fp32" and rng.random() < 0.7
        c["read"] = "state" if c["storage"] == "fp32" and rng.random() < 0.5 else "fields"
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _boxes(case):
    """(nx, ny, nz) of every box of a case."""
    c = _full(case)
    if c["boxes"] == 1:
        return [(c["nx"], c["ny"], c["nz"])]
    r = np.random.RandomState(c["box_seed"] % 2 ** 32)
    return [tuple(int(v) for v in r.randint(c["lmin"], c["lmax"] + 1, 3))
            for _ in range(c["boxes"])]


def _params(c, n):
    """The physical parameters of one box: the phases have equal pressures at
    their reference densities, the lighter one c_s^2 = 1/3."""
    two = c["lattice"] == "d2q9"
    xi, light = (0.6, 4.0 / 9.0) if two else (9.0 / 19.0, 8.0 / 27.0)
    g = c["gamma"]
    heavy = 1.0 - (1.0 - light) / g
    p = dict(nx=n[0], ny=n[1], nz=n[2], rho0_r=1.0, rho0_b=1.0 / g, alpha_r=heavy, alpha_b=light,
             nu_r=(c["tau"] - 0.5) * xi * (1.0 - heavy), nu_b=(c["tau"] - 0.5) * xi * (1.0 - light),
             sigma=c["sigma"] / g, beta=0.7, model=c["model"],
             omega_hi=(c["rate"],) * 9)
    if c["flow"] == "collision":
        p["walls"] = 3
    if c["flow"] == "layer":
        # (the heavy phase lies below; gravity points the unstable way)
        p.update(walls=2, gravity=(0.0, 0.0, -0.04 ** 2 / n[0]), rho_ref=0.5 * (1.0 + 1.0 / g))
    return p


def _inputs(case, seed):
    """Per box: parameters and the initial densities and velocity, float32
    tensors on the GPU of shape (nz, ny, nx) and (3, nz, ny, nx)."""
    c = _full(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = np.random.RandomState(seed % 2 ** 32)
    out = []
    for n in _boxes(case):
        p = _params(c, n)
        nx, ny, nz = n
        z, y, x = (torch.arange(m, device="cuda", dtype=torch.float32).reshape(s) for m, s in
                   ((nz, (-1, 1, 1)), (ny, (1, -1, 1)), (nx, (1, 1, -1))))
        at = rng.uniform(0.0, 1.0, 3)
        u = torch.empty((3, nz, ny, nx), device="cuda")

        def ball(centre, r, wrap=True):
            d2 = 0.0
            for a, q, m in zip((x, y, z), centre, n):
                d = (a - float(q)).abs()
                d = torch.minimum(d, m - d) if wrap else d
                d2 = d2 + d * d
            return (d2 <= r * r).expand(nz, ny, nx)

        small = min(nx, ny) if nz == 1 else min(n)
        if c["flow"] == "droplet":
            red = ball(at * n, c["radius"] * small)
            way = rng.uniform(0.4, 1.0, 3) * rng.choice((-1.0, 1.0), 3)
            way *= c["speed"] / np.linalg.norm(way)
            for a in range(3):
                u[a] = float(way[a])
        elif c["flow"] == "field":
            pitch = 128.0
            bx, by = max(1, int(nx / pitch)), max(1, int(ny / pitch))
            ax, ay = nx / bx, ny / by
            jx = torch.from_numpy(rng.uniform(-0.1, 0.1, (by, bx)).astype(np.float32)).cuda()
            jy = torch.from_numpy(rng.uniform(-0.1, 0.1, (by, bx)).astype(np.float32)).cuda()
            ix, iy = (x / ax).long().clamp(max=bx - 1), (y / ay).long().clamp(max=by - 1)
            dx = x - (ix + 0.5 + jx[iy, ix]) * ax
            dy = y - (iy + 0.5 + jy[iy, ix]) * ay
            red = (dx * dx + dy * dy <= (0.36 * min(ax, ay, pitch)) ** 2).expand(nz, ny, nx)
            way = rng.uniform(0.5, 1.0, 2) * rng.choice((-1.0, 1.0), 2)
            u[0], u[1], u[2] = float(0.03 * way[0]), float(0.03 * way[1]), 0.0
        elif c["flow"] == "collision":
            r = c["radius"] * small
            mid = [(m - 1) / 2.0 + 2.0 * (q - 0.5) for m, q in zip(n, at)]
            left = ball((mid[0] - 2 * r, mid[1], mid[2]), r, False)
            right = ball((mid[0] + 2 * r, mid[1], mid[2]), r, False)
            red = left | right
            u.zero_()
            u[0] = c["speed"] * (left.float() - right.float())
        else:
            h = 0.05 * nx * (torch.cos(2 * math.pi * (x / nx + at[0])) +
                             torch.cos(2 * math.pi * (y / ny + at[1])))
            red = (z < (nz - 1) / 2.0 + h).expand(nz, ny, nx)
            u.zero_()
        noise = 1e-5 * (2.0 * torch.rand(u.shape, device="cuda", generator=gen) - 1.0)
        if nz == 1:
            noise[2] = 0.0
        rr = torch.where(red, p["rho0_r"], 0.0).float().contiguous()
        rb = torch.where(red, 0.0, p["rho0_b"]).float().contiguous()
        out.append((p, rr, rb, u + noise))
    return out


def prepare(case, seed):
    c = _full(case)
    boxes = _inputs(case, seed)
    sim = pkg.Simulation([pkg.box_params(**b[0]) for b in boxes],
                         [b[1].cpu().numpy() for b in boxes], [b[2].cpu().numpy() for b in boxes],
                         [b[3].cpu().numpy() for b in boxes], storage=STORAGE[c["storage"]],
                         lattice=c["lattice"], inplace=c["inplace"])
    if c["schedule"] != "default" and not c["inplace"]:
        sim.autotune(reps=5)
        if c["schedule"] == "compact":
            sim.set_schedule(2)
            sim.set_resident(c["resident"])
    return {"sim": sim, "case": c, "boxes": _boxes(case)}


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _state(sim, c, boxes):
    """The stored populations of every box, views of the state buffer."""
    s = sim.state_tensor().view(torch.float32)
    if c["lattice"] == "d2q9":
        s = s[:18 * sim.total].view(9, sim.total, 2)
    elif c["storage"] == "fp32_pairs":
        s = s[:54 * sim.total].view(27, sim.total, 2)
    else:
        s = s[:54 * sim.total].view(54, sim.total)
    return [s[:, sim.offsets[b]:sim.offsets[b] + n[0] * n[1] * n[2]] for b, n in enumerate(boxes)]


def run(state):
    sim, c = state["sim"], state["case"]
    if c["steps"]:
        sim.step(c["steps"])
    if c["read"] == "state":
        return _state(sim, c, state["boxes"])
    if c["read"] == "monitor":
        return {"diag": sim.reduce_device(), "fields": sim.moments(0, FIELDS)}
    names = ("rho_r", "rho_b", "ux", "uy") if c["lattice"] == "d2q9" else \
        ("rho_r", "rho_b", "ux", "uy", "uz")
    return sim.moments(0, names)


def work(case):
    """A step reads the state once and writes the next state once: the
    populations as stored or, where the schedule keeps the compact state, its
    17 values (and the two FP64 densities of the mass-exact formats).  A
    read-out reads the stored populations once and writes what it returns.
    Operations: about 900 per node and step in three dimensions (moments, the
    stencils, collision, back-transform, recolouring), 250 in two."""
    c = _full(case)
    nodes = sum(a * b * d for a, b, d in _boxes(case))
    two = c["lattice"] == "d2q9"
    moving = 8 if two else 26
    plain = c["storage"] in ("fp32", "fp32_pairs")
    word = 2 if c["storage"] in ("fp16", "bf16", "fp16c", "bf16c") else 4
    pops = 2 * (moving + 1) * 4 if plain else 2 * moving * word + 16
    if c["storage"] in ("fp16c", "bf16c"):
        pops += 2
    step = 2 * pops
    if c["schedule"] == "compact":
        step = 2 * (17 * 4 + (0 if plain else 16))
    b = c["steps"] * step
    if c["schedule"] == "compact" and not c["resident"]:
        b += 2 * pops  # populations in at the start of the call, out at its end
    if c["schedule"] == "compact" and c["resident"]:
        b += pops      # stored for the read-out
    if c["read"] == "monitor":
        b += 2 * pops + 4 * len(FIELDS)
    elif c["read"] == "fields":
        b += pops + 4 * (4 if two else 5)
    per = 250 if two else 900
    return {"bytes": float(b * nodes), "flops": float(per * nodes * max(1, c["steps"]))}


# ---------------------------------------------------------------------------
# The same update in 64 bits, from the definitions
# ---------------------------------------------------------------------------
_C3 = tuple(zip(
    (0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 1, -1, -1, 1),
    (0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 1, -1, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, -1, 1, 1, -1),
    (0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1, 1, -1, -1, 1, 1, -1, 1, -1)))
_C2 = ((0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (1, 1, 0), (-1, -1, 0),
       (1, -1, 0), (-1, 1, 0))


class _Exact:
    """One box: populations of the two colours as lists in velocity order."""

    def __init__(self, p, rr, rb, u, two):
        self.p, self.two, self.dim = p, two, 2 if two else 3
        self.c = _C2 if two else _C3
        self.w = [math.prod((2 / 3 if v == 0 else 1 / 6) for v in c[:self.dim]) for c in self.c]
        xi = 0.6 if two else 9.0 / 19.0
        self.cs2 = (xi * (1 - p["alpha_r"]), xi * (1 - p["alpha_b"]))
        self.shape = rr.shape
        walls = p.get("walls", 0)
        solid = torch.zeros(rr.shape, dtype=torch.bool, device=rr.device)
        if walls & 1:
            solid[:, 0], solid[:, -1] = True, True
        if walls & 2:
            solid[0], solid[-1] = True, True
        self.solid = solid if walls else None
        self.hi = p.get("omega_hi", (1.0,) * 9)
        rr, rb, u = rr.double(), rb.double(), [v.double() for v in u]
        rho, pr = rr + rb, rr * self.cs2[0] + rb * self.cs2[1]
        f = self.equilibrium(rho, pr, u)
        self.pulled = [[(k / rho) * v for v in f] for k in (rr, rb)]

    def at(self, a, c):
        """a(x + c)."""
        return torch.roll(a, (-c[2], -c[1], -c[0]), (0, 1, 2))

    def grad(self, a, axes=(0, 1, 2)):
        g = {d: torch.zeros_like(a) for d in axes if d < self.dim}
        for c, w in zip(self.c[1:], self.w[1:]):
            need = [d for d in g if c[d]]
            if not need:
                continue
            v = self.at(a, c)
            if self.solid is not None:
                v = torch.where(self.at(self.solid, c), a, v)
            for d in need:
                g[d].add_(v, alpha=3.0 * w * c[d])
        return [g.get(d, 0.0) for d in range(3)] if len(axes) > 1 else g.get(axes[0], 0.0)

    # moments about u, one axis at a time; keys (a, b, c) hold orders or
    # velocity components plus one
    def _axes(self, m, u, one):
        for d in range(self.dim):
            new = {}
            for key in m:
                if key[d] != 0:
                    continue
                trip = [m[tuple(i if e == d else k for e, k in enumerate(key))] for i in range(3)]
                for i, v in enumerate(one(*trip, u[d])):
                    new[tuple(i if e == d else k for e, k in enumerate(key))] = v
            m = new
        return m

    def to_moments(self, f, u):
        def one(lo, mid, hi, v):
            return lo + mid + hi, (hi - lo) - v * (lo + mid + hi), \
                hi * (1 - v) ** 2 + mid * v ** 2 + lo * (1 + v) ** 2
        third = 0 if self.two else 1
        return self._axes({(c[0] + 1, c[1] + 1, c[2] + third): f[i] for i, c in enumerate(self.c)},
                          u, one)

    def to_populations(self, k, u):
        def one(k0, k1, k2, v):
            m1 = k1 + v * k0
            m2 = k2 + 2 * v * k1 + v * v * k0
            return (m2 - m1) / 2, k0 - m2, (m2 + m1) / 2
        f = self._axes(k, u, one)
        third = 0 if self.two else 1
        return [f[(c[0] + 1, c[1] + 1, c[2] + third)] for c in self.c]

    def keys(self):
        r = range(3)
        return [(a, b, c) for a in r for b in r for c in (r if not self.two else (0,))]

    def eq_moments(self, rho, pr, u):
        """Central moments of the equilibrium: the generalized one (even
        orders only, independent of u), or the standard one's, from its
        populations."""
        if self.p["model"] == 0:
            return self.to_moments(self.equilibrium(rho, pr, u), u)
        zero = torch.zeros_like(rho)
        k = {}
        for key in self.keys():
            pairs = sum(v == 2 for v in key)
            k[key] = zero if 1 in key else (rho if pairs == 0 else pr / 3.0 ** (pairs - 1))
        return k

    def equilibrium(self, rho, pr, u):
        if self.p["model"] != 0:
            return self.to_populations(self.eq_moments(rho, pr, u), u)
        u2 = sum(v * v for v in u)
        f = []
        for c, w in zip(self.c, self.w):
            cu = sum(c[d] * u[d] for d in range(3) if c[d])
            rest = 3 * w * pr if any(c) else rho - 3 * pr * (1 - self.w[0])
            f.append(rest + w * rho * (3 * cu + 4.5 * cu * cu - 1.5 * u2))
        return f

    def local(self):
        rr, rb = sum(self.pulled[0]), sum(self.pulled[1])
        f = [a + b for a, b in zip(*self.pulled)]
        j = [sum(c[d] * v for c, v in zip(self.c, f) if c[d]) if d < self.dim else
             torch.zeros_like(rr) for d in range(3)]
        if self.solid is not None:
            rr, rb = (torch.where(self.solid, 0.0, v) for v in (rr, rb))
            j = [torch.where(self.solid, 0.0, v) for v in j]
        return rr, rb, f, j

    def interface(self, rr, rb, j):
        p = self.p
        sr, sb = rr / p["rho0_r"], rb / p["rho0_b"]
        den = sr + sb
        phi = torch.where(den > 0, (sr - sb) / torch.where(den > 0, den, 1.0), 0.0)
        g = self.grad(phi)
        mag = sum(v * v for v in g).sqrt()
        live = mag > 1e-12
        if self.solid is not None:
            live = live & ~self.solid
        n = [torch.where(live, v / torch.where(live, mag, 1.0), 0.0) if d < self.dim else
             torch.zeros_like(phi) for d, v in enumerate(g)]
        kap = torch.zeros_like(phi)
        for a in range(self.dim):
            dn = self.grad(n[a])
            kap -= dn[a]
            for b in range(self.dim):
                kap += n[a] * n[b] * dn[b]
        rho = rr + rb
        F = [0.5 * p["sigma"] * kap * torch.where(live, mag, 0.0) * n[d]
             - (rho - p.get("rho_ref", 0.0)) * p.get("gravity", (0.0,) * 3)[d] for d in range(3)]
        safe = torch.where(rho > 0, rho, 1.0)
        u = [(j[d] + 0.5 * F[d]) / safe for d in range(3)]
        if self.solid is not None:
            F = [torch.where(self.solid, 0.0, v) for v in F]
            u = [torch.where(self.solid, 0.0, v) for v in u]
        pr = rr * self.cs2[0] + rb * self.cs2[1]
        return phi, n, F, u, pr, rho, safe

    def step(self):
        """Collide and recolour the pulled populations: the stored state."""
        p, D = self.p, self.dim
        rr, rb, f, j = self.local()
        phi, n, F, u, pr, rho, safe = self.interface(rr, rb, j)
        Q = [-3.0 * self.grad((pr - rho / 3.0) * u[d], (d,)) for d in range(D)]
        nu = 0.5 * ((1 + phi) * p["nu_r"] + (1 - phi) * p["nu_b"])
        w1 = 1.0 / (rho * nu / torch.where(pr > 0, pr, 1.0) + 0.5)
        k, e = self.to_moments(f, u), self.eq_moments(rho, pr, u)
        w0, w3, w4, w5, w6, w7, w8, w9, w10 = self.hi
        s = {}
        axis = [tuple(int(d == a) for d in range(3)) for a in range(3)]
        dbl = [tuple(2 * v for v in a) for a in axis]
        s[(0, 0, 0)] = rho
        for d in range(D):
            s[axis[d]] = (1 - w0) * k[axis[d]] + (1 - w0 / 2) * F[d]
            for b in range(d):
                q = tuple(x + y for x, y in zip(axis[d], axis[b]))
                s[q] = (1 - w1) * k[q]
        tr, sq = sum(k[dbl[d]] for d in range(D)), sum(Q)
        for d in range(D):  # bulk rate 1: the trace relaxes to D p
            s[dbl[d]] = (D * pr + 0.5 * sq) / D + (1 - w1) * (k[dbl[d]] - tr / D) \
                + (1 - 0.5 * w1) * (Q[d] - sq / D)
            if p["model"] == 0:
                se = sum(e[dbl[a]] for a in range(D))
                s[dbl[d]] = s[dbl[d]] - pr + se / D + w1 * (e[dbl[d]] - se / D)

        def relax(q, w):
            return (1 - w) * k[q] + w * e[q]

        for q in self.keys():  # higher orders, each toward its equilibrium
            if q in s:
                continue
            force = [d for d in range(D) if q[d] == 1]
            pairs = sum(v == 2 for v in q)
            w = {3: w5 if pairs == 0 else None, 4: w8 if pairs == 1 else None,
                 5: w9, 6: w10}[sum(q)]
            if w is None:
                continue
            s[q] = relax(q, w)
            if sum(q) == 5:
                s[q] = s[q] + (1 - w / 2) * F[force[0]] / 3.0 ** pairs
        for d in range(D):  # third order: sums at one rate, differences at another
            qs = [tuple(axis[d][x] + dbl[b][x] for x in range(3)) for b in range(D) if b != d]
            mean_k, mean_e = sum(k[q] for q in qs) / len(qs), sum(e[q] for q in qs) / len(qs)
            for q in qs:
                s[q] = (1 - w3) * mean_k + w3 * mean_e + (1 - w3 / 2) * F[d] / 3.0 \
                    + (1 - w4) * (k[q] - mean_k) + w4 * (e[q] - mean_e)
        fours = [q for q in self.keys() if sum(q) == 4 and 1 not in q]
        mean_k = sum(k[q] for q in fours) / len(fours)
        mean_e = sum(e[q] for q in fours) / len(fours)
        for q in fours:
            s[q] = (1 - w7) * mean_k + w7 * mean_e + (1 - w6) * (k[q] - mean_k) \
                + w6 * (e[q] - mean_e)
        post = self.to_populations(s, u)
        cr, cb = rr / safe, rb / safe
        R = p["beta"] * cr * cb * pr
        stored = [[], []]
        for i, (c, w) in enumerate(zip(self.c, self.w)):
            d = 3.0 * w * R * sum(c[a] * n[a] for a in range(3)) if any(c) else 0.0
            stored[0].append(cr * post[i] + d)
            stored[1].append(cb * post[i] - d)
        if self.solid is not None:  # what arrived at a solid node goes back
            for k2 in range(2):
                for i, c in enumerate(self.c):
                    o = self.c.index(tuple(-v for v in c))
                    stored[k2][i] = torch.where(self.solid, self.pulled[k2][o], stored[k2][i])
        self.stored = stored

    def stream(self):
        self.pulled = [[self.at(v, tuple(-x for x in c)) for v, c in zip(s, self.c)]
                       for s in self.stored]

    def fields(self):
        rr, rb, _, j = self.local()
        phi, _, _, u, pr, _, _ = self.interface(rr, rb, j)
        return dict(rho_r=rr, rho_b=rb, phi=phi, p=pr, ux=u[0], uy=u[1], uz=u[2])

    def diagnostics(self):
        """Masses, momentum, the two pressures, radius, red centroid, kinetic
        energy, count of non-finite nodes (periodic box, its own centre)."""
        f = self.fields()
        rho = f["rho_r"] + f["rho_b"]
        u = [f["ux"], f["uy"], f["uz"]]
        radius = (3 * (0.5 * (1 + f["phi"])).sum() / (4 * math.pi)) ** (1 / 3)
        off = []
        for a, dim in ((0, 2), (1, 1), (2, 0)):
            m = self.shape[dim]
            d = torch.arange(m, device=rho.device, dtype=torch.float64) - 0.5 * (m - 1)
            off.append(d.reshape([-1 if e == dim else 1 for e in range(3)]))
        dist = (off[0] ** 2 + off[1] ** 2 + off[2] ** 2).sqrt()
        inside, outside = dist < radius - 3, dist > radius + 5
        mass = f["rho_r"].sum()
        out = [mass, f["rho_b"].sum()] + [(rho * v).sum() for v in u]
        out += [f["p"][inside].mean(), f["p"][outside].mean(), radius]
        out += [(f["rho_r"] * d).sum() / mass for d in off]
        out += [(0.5 * rho * (u[0] ** 2 + u[1] ** 2 + u[2] ** 2)).sum(), torch.zeros_like(mass)]
        return torch.stack(out).reshape(1, -1)


def exact(case, seed):
    c = _full(case)
    nodes = sum(a * b * d for a, b, d in _boxes(case))
    if nodes * max(1, c["steps"]) > 3.5e8:
        return None
    out = []
    for p, rr, rb, u in _inputs(case, seed):
        sim = _Exact(p, rr, rb, u, c["lattice"] == "d2q9")
        for k in range(c["steps"]):
            sim.step()
            if k + 1 < c["steps"] or c["read"] != "state":
                sim.stream()
        if c["read"] == "fields":
            f = sim.fields()
            return {k: f[k] for k in f if k in ("rho_r", "rho_b", "ux", "uy") or
                    (k == "uz" and not sim.two)}
        if c["read"] == "monitor":
            return {"diag": sim.diagnostics(), "fields": sim.fields()}
        flat = [[v.reshape(-1) for v in s] for s in sim.stored]
        if c["lattice"] == "d2q9" or c["storage"] == "fp32_pairs":
            out.append(torch.stack([torch.stack((a, b), -1) for a, b in zip(*flat)]))
        else:
            out.append(torch.stack(flat[0] + flat[1]))
        del sim, flat
    return out
