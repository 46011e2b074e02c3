"""Timed workloads of the FAM library: what one pass of each is, its inputs, its necessary work and its 64-bit value.

A case is one use of the public entry points (Fam.run, Fam.step, fam_step_static, a batched context,
Fam.adjoint, evolve) on a mesh: the smallest are the accuracy-table meshes, where a step is a handful of
tiny launches; the largest are 2048 x 2048.  ``exact`` evaluates the same steps with plain torch in 64 bits
(reconstruction weights from solving the moment systems numerically, point values by matrix products).
"""
import math

import numpy as np
import torch

GAMMA = 1.4
BATCH_SIZES = (64, 96, 128, 192, 256, 384, 512)


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _case(kind, init, nx, ny, k, steps, **kw):
    """kind: run | step | static | batch | adjoint | evolve; init: the initial data (``_state``).
    t_final > 0: a run to that time instead of a step count.  tuned: the launch shapes are autotuned."""
    c = dict(kind=kind, init=init, dim=1 if ny == 1 else 2, nx=nx, ny=ny, k=k, steps=steps, t_final=0.0,
             system="euler", bc="periodic", oe="type2", pp=False, dmr=False, char=False, dt_rule=0, cfl=0.2,
             tuned=False, every=0, sizes="")
    c.update(kw)
    return c


def listed():
    quad = dict(bc="transmissive", pp=True)
    return [
        # the 1D accuracy tables: a few hundred cells at most, thousands of steps, each a few tiny launches
        _case("run", "burgers", 120, 1, 5, 0, name="burgers1d-n120", system="burgers", dt_rule=1, cfl=0.1,
              t_final=0.02),
        # the shock / density-wave problem at its full 4000 cells
        _case("run", "shock1d", 4000, 1, 5, 200, name="shock1d-n4000", bc="transmissive"),
        # the 2D accuracy tables (N = 20..120), run to a time
        _case("run", "diagonal", 40, 40, 4, 0, name="smooth2d-n40-k4", dt_rule=1, cfl=0.1, t_final=0.02),
        # a program that steps by itself and reads the time step of every step: latency of single calls
        _case("step", "quadrant", 96, 80, 5, 10, name="step-96x80", **quad),
        # the allocation-free step on a small ragged mesh
        _case("static", "waves", 203, 131, 5, 10, name="static-203x131"),
        # a mid-size shock problem with the default launch shapes
        _case("run", "quadrant", 256, 256, 5, 20, name="quadrant-256", **quad),
        # a scalar law with Type I elimination (global statistics in every step)
        _case("run", "scalar", 700, 555, 4, 20, name="burgers2d-700x555-type1", system="burgers", oe="type1"),
        # the double Mach reflection at its published size and CFL number
        _case("run", "mach", 1440, 480, 5, 20, name="mach-1440x480", pp=True, dmr=True, cfl=0.55, tuned=True),
        # the headline problem
        _case("run", "quadrant", 2048, 2048, 5, 12, name="quadrant-2048", tuned=True, **quad),
        # the highest order without the limiter
        _case("run", "waves", 1201, 1000, 6, 10, name="waves-1201x1000-k6", tuned=True),
        # many uneven meshes in one context
        _case("batch", "quadrant", 512, 512, 5, 10, name="batch-40", tuned=True, sizes=_sizes(40, np.random.default_rng(1)),
              **quad),
        # gradient of the window functional through the checkpointed adjoint
        _case("adjoint", "noisy", 512, 512, 5, 12, name="adjoint-512", every=4),
    ]


def _sizes(count, rng):
    return ",".join(str(int(s)) for s in rng.choice(BATCH_SIZES, size=count))


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def steps(cells, most):
        # a pass of a few milliseconds up to about the largest listed one's half
        return max(4, min(most, int(rng.uniform(0.4, 1.0) * 2.4e7 / cells)))

    kind = rng.choice(["run1d", "run1d", "table2d", "quadrant", "quadrant", "waves", "scalar", "mach", "step", "static",
                       "batch", "adjoint", "evolve"])
    k = rng.choice([3, 4, 5, 5, 5, 6])
    if kind == "run1d":
        if rng.random() < 0.5:
            n = size(30, 800)
            sys_ = rng.choice(["burgers", "advection", "euler"])
            return _case("run", "burgers" if sys_ != "euler" else "diagonal", n, 1, k, rng.randrange(60, 240),
                         system=sys_, dt_rule=1, cfl=0.1, oe=rng.choice(["type2", "type2", "type1", "off"]))
        n = 10 * size(40, 600)   # the shock on a cell face
        char = rng.random() < 0.3
        return _case("run", "shock1d", n, 1, 5 if char else max(k, 5), rng.randrange(60, 240), bc="transmissive", char=char)
    if kind == "table2d":
        n = size(20, 120)
        return _case("run", "diagonal", n, n, k, rng.randrange(10, 60), dt_rule=1, cfl=0.1)
    if kind == "quadrant":
        nx = size(64, 2048)
        ny = max(60, min(2048, int(nx * rng.uniform(0.5, 1.5))))
        return _case("run", "quadrant", nx, ny, k, steps(nx * ny, 40), bc="transmissive", pp=True,
                     tuned=rng.random() < 0.5)
    if kind == "waves":
        nx, ny = size(150, 1600), size(150, 1600)
        return _case("run", "waves", nx, ny, k, steps(nx * ny, 40), tuned=rng.random() < 0.5,
                     oe=rng.choice(["type2", "type2", "off"]))
    if kind == "scalar":
        nx, ny = size(100, 1500), size(100, 1500)
        return _case("run", "scalar", nx, ny, k, steps(nx * ny, 40), system=rng.choice(["burgers", "advection"]),
                     oe=rng.choice(["type1", "type2"]), bc=rng.choice(["periodic", "transmissive"]))
    if kind == "mach":
        ny = size(60, 500)
        char = rng.random() < 0.4
        return _case("run", "mach", 3 * ny + rng.randrange(4), ny, 5 if char else k, steps(3 * ny * ny, 40), pp=True,
                     dmr=True, cfl=0.5, char=char, tuned=rng.random() < 0.5)
    if kind == "step":
        nx, ny = size(40, 400), size(40, 400)
        return _case("step", "quadrant", nx, ny, k, rng.randrange(4, 12), bc="transmissive", pp=True)
    if kind == "static":
        nx, ny = size(40, 500), size(40, 500)
        return _case("static", "waves", nx, ny, k, rng.randrange(4, 12))
    if kind == "batch":
        n = rng.randrange(6, 64)
        sizes = ",".join(str(rng.choice(BATCH_SIZES)) for _ in range(n))
        return _case("batch", "quadrant", 512, 512, 5, rng.randrange(4, 8), bc="transmissive", pp=True, tuned=True,
                     sizes=sizes)
    nx, ny = size(48, 640), size(48, 640)
    n = rng.randrange(4, 12)
    return _case(kind, "noisy", nx, ny, k, n, every=rng.randrange(2, n + 1))


# ---------------------------------------------------------------------------
# inputs: moments of seeded initial data by a 6-point Gauss rule per direction
# ---------------------------------------------------------------------------
def _box(c):
    if c["init"] == "shock1d":
        return -5.0, 5.0, 0.0, 1.0
    if c["init"] in ("burgers", "diagonal"):
        return 0.0, 2.0, 0.0, 2.0
    if c["init"] == "mach":
        return 0.0, 3.0, 0.0, 1.0
    return 0.0, 1.0, 0.0, 1.0


def _prim(init, system, rng):
    """Initial data as a function of (x, y): scalar u, or (rho, u, v, p) of the Euler equations."""
    one = torch.ones_like
    if init == "burgers" or (init == "scalar" and system != "euler"):
        a, ph = rng.uniform(0.3, 0.6), rng.uniform(0.0, 2.0 * math.pi)
        w = math.pi if init == "burgers" else 2.0 * math.pi
        return lambda x, y: (a + torch.sin(w * x + ph) * (torch.cos(w * y) if init == "scalar" else 1.0),)
    if init == "diagonal":
        ph = rng.uniform(0.0, 2.0 * math.pi)
        return lambda x, y: (1.0 + 0.2 * torch.sin(math.pi * (x + y) + ph), one(x), one(x), one(x))
    if init == "shock1d":
        # the Mach 3 shock meeting a density wave, in a frame moving at du
        ph, du = rng.uniform(0.0, 2.0 * math.pi), rng.uniform(0.05, 0.2)
        return lambda x, y: (torch.where(x < -4.0, 3.857143 * one(x), 1.0 + 0.2 * torch.sin(5.0 * x + ph)),
                             torch.where(x < -4.0, (2.629369 + du) * one(x), du * one(x)), 0.0 * x,
                             torch.where(x < -4.0, 10.33333 * one(x), one(x)))
    if init == "quadrant":
        st = [(rng.uniform(0.2, 1.5), rng.uniform(-0.7, 0.7), rng.uniform(-0.7, 0.7), rng.uniform(0.1, 1.5))
              for _ in range(4)]

        def f(x, y):
            pick = [torch.where(x > 0.5, st[0][q], st[1][q]) for q in range(4)]
            low = [torch.where(x > 0.5, st[3][q], st[2][q]) for q in range(4)]
            return tuple(torch.where(y > 0.5, a, b).to(x.dtype) for a, b in zip(pick, low))
        return f
    if init == "mach":
        # gas ahead of the shock weakly disturbed (a uniform one keeps a component at rounding level)
        ph = rng.uniform(0.0, 2.0 * math.pi, size=4)

        def f(x, y):
            post = x < 1.0 / 6.0 + y / math.sqrt(3.0)
            d = [0.02 * torch.sin(2.0 * math.pi * (x + (1 + q) * y) + ph[q]) for q in range(4)]
            ahead = (1.4 + d[0], 0.1 + d[1], 0.1 + d[2], 1.0 + d[3])
            back = (8.0, 8.25 * math.cos(math.pi / 6), -8.25 * math.sin(math.pi / 6), 116.5)
            return tuple(torch.where(post, b * one(x), a) for a, b in zip(ahead, back))
        return f
    # waves: four density modes carried by a uniform flow (noisy: with cell noise, see _state)
    amp, ks, ph = rng.uniform(-0.25, 0.25, 4), rng.integers(1, 4, size=(4, 2)), rng.uniform(0.0, 2.0 * math.pi, 4)
    sg = rng.choice([-1.0, 1.0], 4)
    return lambda x, y: (1.0 + 0.2 * sum(amp[m] * torch.sin(2.0 * math.pi * (ks[m][0] * x + sg[m] * ks[m][1] * y) + ph[m])
                                         for m in range(4)), 0.5 * one(x), 0.5 * one(x), one(x))


def _state(c, seed, dev, nx=None, ny=None):
    """The moment state [component, moment, (ny,) nx] of the case's initial data."""
    nx, ny = nx or c["nx"], ny or c["ny"]
    f = _prim(c["init"], c["system"], np.random.default_rng(seed))
    x0, x1, y0, y1 = _box(c)
    q, w = np.polynomial.legendre.leggauss(6)
    q, w = 0.5 * q, 0.5 * w
    dx, dy = (x1 - x0) / nx, (y1 - y0) / ny
    xc = x0 + (torch.arange(nx, dtype=torch.float64, device=dev) + 0.5) * dx
    yc = y0 + (torch.arange(ny, dtype=torch.float64, device=dev) + 0.5) * dy
    out = None
    for b in range(6) if c["dim"] == 2 else (0,):
        for a in range(6):
            X = (xc + dx * q[a])[None, :].expand(ny, nx)
            Y = ((yc + dy * q[b]) if c["dim"] == 2 else torch.zeros_like(yc))[:, None].expand(ny, nx)
            wt = w[a] * (w[b] if c["dim"] == 2 else 1.0)
            u = _conserved(f(X, Y), c)
            m = torch.stack([u, q[a] * u] + ([q[b] * u] if c["dim"] == 2 else []), dim=1) * wt
            out = m if out is None else out.add_(m)
    if c["init"] == "noisy":
        # one percent of noise from cell to cell, as measured data has it; it also keeps every interface jump
        # away from zero, where the gradient of its magnitude is one-sided
        g = torch.Generator(device=dev).manual_seed(int(seed))
        r = torch.rand(out.shape, dtype=torch.float64, device=dev, generator=g) - 0.5
        out[:, 0] *= 1.0 + 0.02 * r[:, 0]
        out[:, 1:] += 0.004 * r[:, 1:] * out[:, :1]
    return (out if c["dim"] == 2 else out[:, :, 0, :]).contiguous()


def _conserved(v, c):
    if c["system"] != "euler":
        return v[0][None]
    r, u, w, p = v
    if c["dim"] == 1:
        return torch.stack([r, r * u, p / (GAMMA - 1.0) + 0.5 * r * u * u])
    return torch.stack([r, r * u, r * w, p / (GAMMA - 1.0) + 0.5 * r * (u * u + w * w)])


def _meshes(c):
    return [(int(s), int(s)) for s in c["sizes"].split(",")] if c["kind"] == "batch" else [(c["nx"], c["ny"])]


def _fixed_dt(c):
    """Time step of the gradient cases: half the CFL step of the waves (speed at most 1/2 + sqrt(1.4/0.7))."""
    a = 0.5 + math.sqrt(GAMMA / 0.7)
    return 0.5 * c["cfl"] / (a * c["nx"] + a * c["ny"])


# ---------------------------------------------------------------------------
# a user's program
# ---------------------------------------------------------------------------
def _config(c, nx, ny):
    from paper_2609_26194_amd import FamConfig
    x0, x1, y0, y1 = _box(c)
    return FamConfig(dim=c["dim"], nx=nx, ny=ny, x0=x0, x1=x1, y0=y0, y1=y1, k=c["k"], system=c["system"], gamma=GAMMA,
                     a=(1.0, 0.5), bc_x=c["bc"], bc_y=c["bc"], oe=c["oe"], cfl=c["cfl"], pp=c["pp"],
                     dt_rule=c["dt_rule"], dmr=c["dmr"], char_vars=c["char"])


def prepare(case, seed):
    from paper_2609_26194_amd import Fam
    c = case
    dev = torch.device("cuda")
    cfgs = [_config(c, nx, ny) for nx, ny in _meshes(c)]
    parts = [_state(c, seed + 1000 * i, dev, nx, ny) for i, (nx, ny) in enumerate(_meshes(c))]
    s = {"c": c, "cfg": cfgs[0]}
    if c["kind"] == "batch":
        s["U0"] = torch.cat([p.reshape(-1) for p in parts])
        s["fam"] = Fam(None, batch=cfgs)
    else:
        s["U0"] = parts[0]
        if c["kind"] != "static":
            s["fam"] = Fam(cfgs[0])
    if c["tuned"]:
        s["fam"].autotune(s["U0"])
    if c["kind"] == "evolve":
        g = torch.Generator(device=dev).manual_seed(int(seed))
        s["weight"] = torch.randn(s["U0"].shape, dtype=torch.float64, device=dev, generator=g)
        s["U0"].requires_grad_(True)
    elif c["kind"] != "adjoint":
        s["U"] = torch.empty_like(s["U0"])
        s["dts"] = torch.zeros(max(1, c["steps"]), dtype=torch.float64, device=dev)
    return s


def run(s):
    """One pass: from the initial data, through the steps (and back, for a gradient)."""
    c = s["c"]
    if c["kind"] == "adjoint":
        J, g = s["fam"].adjoint(s["U0"], c["steps"], _fixed_dt(c), c["every"])
        return {"J": J, "grad": g}
    if c["kind"] == "evolve":
        from paper_2609_26194_amd.autograd import evolve
        U = evolve(s["fam"], s["U0"], c["steps"], _fixed_dt(c), c["every"])
        (g,) = torch.autograd.grad(U, s["U0"], s["weight"])
        return {"U": U.detach(), "grad": g}
    U = s["U"]
    U.copy_(s["U0"])
    if c["kind"] == "step":
        for n in range(c["steps"]):
            s["fam"].step(U, dt_used=s["dts"][n:n + 1])
        return {"U": U, "dt": s["dts"]}
    if c["kind"] == "static":
        from paper_2609_26194_amd.fam import fam_step_static
        stream = torch.cuda.current_stream().cuda_stream
        for n in range(c["steps"]):
            fam_step_static(s["cfg"], stream, U, dt_used=s["dts"][n:n + 1])
        return {"U": U, "dt": s["dts"]}
    if c["dmr"]:
        s["fam"].set_time(0.0)
    if c["t_final"] > 0.0:
        s["fam"].set_time(0.0)
        n, t = s["fam"].run(U, c["t_final"], 0)
        return {"U": U, "steps": n, "t": t}
    n, _ = s["fam"].run(U, 0.0, c["steps"])
    return {"U": U, "steps": n}


# ---------------------------------------------------------------------------
# necessary work
# ---------------------------------------------------------------------------
def _steps_of(c):
    """Steps of a pass; for a run to a time, from the largest speed its data can have."""
    if c["t_final"] <= 0.0:
        return c["steps"]
    h = lambda n: (2.0 / n) ** (c["k"] / 3.0)
    a = 1.6 if c["system"] == "burgers" else 1.0 + math.sqrt(GAMMA / 0.8)
    rate = a / h(c["nx"]) + (a / h(c["ny"]) if c["dim"] == 2 else 0.0)
    return int(c["t_final"] * rate / c["cfl"]) + 1


def work(case):
    """One state read and one written per pass (a gradient reads the cotangent and writes the gradient too);
    operations of the algorithm per cell and step: reconstruction, point values, fluxes, quadrature, elimination."""
    from paper_2609_26194_amd.opcount import oe_flops, stage_flops
    c = case
    nc = 1 if c["system"] != "euler" else c["dim"] + 2
    cells = sum(nx * ny for nx, ny in _meshes(c))
    values = cells * nc * (3 if c["dim"] == 2 else 2)
    if c["dim"] == 2:
        per = 3 * stage_flops(c["k"], nc) + (oe_flops(c["k"], nc) if c["oe"] != "off" else 0)
    else:
        per = 3 * (nc * (6 * c["k"] + 6 * 2 * c["k"] + 40) + 6 * 12) + nc * 40 + 40
    grad = c["kind"] in ("adjoint", "evolve")
    # reverse mode: the forward and about three times its operations
    return {"bytes": 8.0 * values * (4 if grad else 2), "flops": float(per) * cells * _steps_of(c) * (4 if grad else 1)}


# ---------------------------------------------------------------------------
# the same steps in plain torch, 64 bits
# ---------------------------------------------------------------------------
_NODE = [0.5 * math.sqrt(3.0 / 7.0 + s * 2.0 / 7.0 * math.sqrt(6.0 / 5.0)) for s in (1.0, -1.0)]
NODES = [-_NODE[0], -_NODE[1], _NODE[1], _NODE[0]]
WEIGHTS = [(18.0 - math.sqrt(30.0)) / 72.0, (18.0 + math.sqrt(30.0)) / 72.0] * 2
WEIGHTS[2], WEIGHTS[3] = WEIGHTS[1], WEIGHTS[0]


def _leg(m, t):
    """Scaled Legendre polynomial of degree m on [-1/2, 1/2] (any positive scaling spans the same space)."""
    return np.polynomial.legendre.Legendre.basis(m)(2.0 * np.asarray(t, dtype=np.float64))


def _operators(dim, k):
    """(stencil slots, {point set: matrix}): each slot is (x offset, y offset, moment); a matrix maps the
    stencil values to point values of p_k, the projection onto degree k - 1 of the polynomial that matches
    the slots' moments (products of Legendre polynomials are orthogonal, so projecting is truncating)."""
    if dim == 1:
        slots = [(a, 0, 0) for a in (-1, 0, 1)] + [(a, 0, 1) for a in ((0,) if k <= 4 else (-1, 0, 1))]
        space = [(p, 0) for p in range(len(slots))]
    else:
        slots = [(a, b, 0) for b in (-1, 0, 1) for a in (-1, 0, 1)]
        if k <= 4:
            slots += [(0, 0, 1), (0, 0, 2)]
            space = [(p, t - p) for t in range(4) for p in range(t + 1)] + [(2, 2)]
        else:
            slots += [(a, b, 1) for b in (-1, 0, 1) for a in (-1, 0, 1) if not (a == 0 and b != 0)]
            slots += [(a, b, 2) for b in (-1, 0, 1) for a in (-1, 0, 1) if not (b == 0 and a != 0)]
            space = [(p, t - p) for t in range(6) for p in range(t + 1)] + [(4, 2), (2, 4)]
    q, w = np.polynomial.legendre.leggauss(8)
    q, w = 0.5 * q, 0.5 * w
    one = lambda m, o, kind: float(np.sum(w * _leg(m, q + o) * (q if kind else 1.0)))
    A = np.array([[one(p, a, kind == 1) * one(r, b, kind == 2) for p, r in space] for a, b, kind in slots])
    keep = [n for n, (p, r) in enumerate(space) if p + r <= k - 1]
    R = np.linalg.inv(A)[keep]
    if dim == 1:
        sets = {"faces": [(0.5, 0.0), (-0.5, 0.0)], "flux": [(0.5, 0.0), (-0.5, 0.0)] + [(x, 0.0) for x in NODES]}
    else:
        sets = {"faces": [(0.5, 0.0), (-0.5, 0.0), (0.0, 0.5), (0.0, -0.5)],
                "flux": [(s, e) for s in (0.5, -0.5) for e in NODES] + [(e, s) for s in (0.5, -0.5) for e in NODES] +
                        [(NODES[a], NODES[b]) for b in range(4) for a in range(4)]}
    mats = {}
    for name, pts in sets.items():
        E = np.array([[float(_leg(space[n][0], x)) * float(_leg(space[n][1], y)) for n in keep] for x, y in pts])
        mats[name] = E @ R
    return slots, mats


class _Exact:
    """The scheme on [component, moment, ny, nx] tensors (ny = 1 in 1D)."""

    def __init__(self, c, nx, ny, dev):
        self.c, self.nx, self.ny, self.dim, self.dev = c, nx, ny, c["dim"], dev
        x0, x1, y0, y1 = _box(c)
        self.x0, self.y1 = x0, y1
        self.dx, self.dy = (x1 - x0) / nx, (y1 - y0) / ny
        self.slots, mats = _operators(self.dim, c["k"])
        self.mats = {n: torch.tensor(m, dtype=torch.float64, device=dev) for n, m in mats.items()}
        self.gk = {1: 25.0, 2: 25.0}[self.dim] if c["k"] <= 4 else (12.5 if self.dim == 1 else 15.0)
        self.euler = c["system"] == "euler"

    # physics -----------------------------------------------------------
    def pressure(self, u):
        return (GAMMA - 1.0) * (u[-1] - 0.5 * sum(m * m for m in u[1:-1]) / u[0])

    def flux(self, u, d):
        if self.c["system"] == "advection":
            return (1.0, 0.5)[d] * u
        if self.c["system"] == "burgers":
            return 0.5 * u * u
        p, v = self.pressure(u), u[1 + d] / u[0]
        out = [u[1 + d]] + [u[m] * v + (p if m == 1 + d else 0.0) for m in range(1, len(u) - 1)] + [(u[-1] + p) * v]
        return torch.stack(out)

    def speed(self, u, d):
        if self.c["system"] == "advection":
            return torch.full_like(u[0], (1.0, 0.5)[d])
        if self.c["system"] == "burgers":
            return u[0].abs()
        return (u[1 + d] / u[0]).abs() + torch.sqrt(GAMMA * self.pressure(u) / u[0])

    # ghost cells, stencils ---------------------------------------------
    def pad(self, U, t):
        g = 2

        def index(n, per):
            i = torch.arange(-g, n + g, device=self.dev)
            return i % n if per else i.clamp(0, n - 1)
        per = self.c["bc"] == "periodic" and not self.c["dmr"]
        P = U[..., index(self.nx, per)]
        if self.dim == 1:
            return P
        P = P[..., index(self.ny, per), :]
        return self.mach_ghosts(U, P, t) if self.c["dmr"] else P

    def mach_ghosts(self, U, P, t):
        def const(r, u, v, p):
            q = [r, r * u, r * v, p / (GAMMA - 1.0) + 0.5 * r * (u * u + v * v)]
            return torch.tensor([[[[a]], [[0.0]], [[0.0]]] for a in q], dtype=torch.float64, device=self.dev)
        post = const(8.0, 8.25 * math.cos(math.pi / 6), -8.25 * math.sin(math.pi / 6), 116.5)
        pre = const(1.4, 0.0, 0.0, 1.0)
        x = self.x0 + (torch.arange(-2, self.nx + 2, device=self.dev, dtype=torch.float64) + 0.5) * self.dx
        P = P.clone()
        P[..., 2:-2, :2] = post
        P[..., -2:, :] = torch.where(x < 1.0 / 6.0 + (self.y1 + 20.0 * t) / math.sqrt(3.0), post, pre)
        sign = torch.ones(4, 3, 1, 1, dtype=torch.float64, device=self.dev)
        sign[:, 2] = -1.0          # the wall mirrors eta ...
        sign[2] = -sign[2]         # ... and the normal momentum
        cols = torch.arange(-2, self.nx + 2, device=self.dev).clamp(0, self.nx - 1)
        wall = (U[..., :2, :].flip(-2) * sign)[..., cols]
        P[..., :2, :] = torch.where(x < 1.0 / 6.0, post, wall)
        return P

    def points(self, P, name):
        """Point values [component, point, ny (+ 2), nx + 2] on the interior cells and their ring."""
        H, W = (P.shape[-2] - 2, P.shape[-1] - 2) if self.dim == 2 else (1, P.shape[-1] - 2)
        o = 1 if self.dim == 2 else 0
        S = torch.stack([P[:, m, o + b: o + b + H, 1 + a: 1 + a + W] for a, b, m in self.slots])
        V = self.mats[name] @ S.reshape(len(self.slots), -1)
        return V.reshape(-1, P.shape[0], H, W).transpose(0, 1)

    def limit(self, V, avg):
        """Scaling limiter: density, then pressure, kept above min(1e-13, rho, p) at every flux point."""
        eps = torch.clamp(torch.minimum(avg[0], self.pressure(avg)), max=1e-13)
        lo = V[0].min(dim=0).values
        t1 = torch.where(lo < eps, (avg[0] - eps) / torch.where(lo < eps, avg[0] - lo, 1.0), 1.0)
        A = avg[:, None]
        w = torch.cat([A[:1] + t1 * (V[:1] - A[:1]), V[1:]])
        d = w - A
        kk = 2.0 / (GAMMA - 1.0)
        a = 2.0 * d[0] * d[3] - d[1] ** 2 - d[2] ** 2
        b = 2.0 * (A[0] * d[3] + d[0] * A[3]) - 2.0 * (A[1] * d[1] + A[2] * d[2]) - kk * eps * d[0]
        e = 2.0 * A[0] * A[3] - A[1] ** 2 - A[2] ** 2 - kk * eps * A[0]
        s = torch.sqrt(torch.clamp(b * b - 4.0 * a * e, min=0.0))
        q = -0.5 * (b + torch.where(b >= 0, s, -s))
        r1 = torch.where(a == 0, 2.0, q / torch.where(a == 0, 1.0, a))
        r2 = e / torch.where(q == 0, 1.0, q)
        ok = lambda r: torch.where((r > 0) & (r <= 1), r, 2.0)
        r = torch.minimum(ok(r1), ok(r2))
        t2 = torch.where((self.pressure(w) < eps) & (r <= 1), r, 1.0).min(dim=0).values
        return torch.where((t1 < 1) | (t2 < 1), A + t2 * (w - A), V)

    # one step ------------------------------------------------------------
    def residual(self, U, t):
        P = self.pad(U, t)
        V = self.points(P, "flux")
        if self.c["pp"]:
            V = self.limit(V, P[:, 0, 1:-1, 1:-1])
        W = torch.tensor(WEIGHTS, dtype=torch.float64, device=self.dev)
        X = torch.tensor(NODES, dtype=torch.float64, device=self.dev)

        def face(L, R, d):
            alpha = torch.max(self.speed(U[:, 0], d))
            return 0.5 * (self.flux(L, d) + self.flux(R, d)) - 0.5 * alpha * (R - L)
        if self.dim == 1:
            F = face(V[:, 0, :, :-1], V[:, 1, :, 1:], 0)
            vol = torch.einsum("q,cqyx->cyx", W, self.flux(V[:, 2:, :, 1:-1], 0))
            return torch.stack([-(F[..., 1:] - F[..., :-1]) / self.dx, (vol - 0.5 * (F[..., 1:] + F[..., :-1])) / self.dx],
                               dim=1)
        F = face(V[:, 0:4, 1:-1, :-1], V[:, 4:8, 1:-1, 1:], 0)
        G = face(V[:, 8:12, :-1, 1:-1], V[:, 12:16, 1:, 1:-1], 1)
        Fb, Ft = (torch.einsum("q,cqyx->cyx", w, F) for w in (W, W * X))
        Gb, Gt = (torch.einsum("q,cqyx->cyx", w, G) for w in (W, W * X))
        W2 = (W[:, None] * W[None, :]).reshape(-1)
        vol = V[:, 16:, 1:-1, 1:-1]
        V1, V2 = (torch.einsum("q,cqyx->cyx", W2, self.flux(vol, d)) for d in (0, 1))
        ddx = lambda f: (f[..., 1:] - f[..., :-1]) / self.dx
        ddy = lambda f: (f[..., 1:, :] - f[..., :-1, :]) / self.dy
        return torch.stack([-ddx(Fb) - ddy(Gb),
                            V1 / self.dx - (Fb[..., 1:] + Fb[..., :-1]) / (2 * self.dx) - ddy(Gt),
                            V2 / self.dy - (Gb[..., 1:, :] + Gb[..., :-1, :]) / (2 * self.dy) - ddx(Ft)], dim=1)

    def eliminate(self, U, dt, t):
        if self.c["oe"] == "off":
            return U
        P = self.pad(U, t)
        V = self.points(P, "faces")
        rows = (-1, 0, 1) if self.dim == 2 else (0,)
        o = 2 if self.dim == 2 else 0
        patch = torch.stack([P[:, 0, o + b: o + b + self.ny, 2 + a: 2 + a + self.nx] for b in rows for a in (-1, 0, 1)],
                            dim=1)
        if self.c["oe"] == "type2":
            D = (patch - patch.sum(dim=1, keepdim=True)).abs().max(dim=1).values
            eps = 1e-14 * torch.clamp(patch.abs().max(dim=1).values, min=1.0)
        else:
            flat = U[:, 0].reshape(U.shape[0], -1)
            D = (flat - flat.mean(dim=1, keepdim=True)).abs().max(dim=1).values[:, None, None]
            eps = 1e-14 * torch.clamp(flat.abs().max(dim=1).values, min=1.0)[:, None, None]
        expo = 0.0
        for d in range(self.dim):
            C = V if self.dim == 1 else (V[:, :, 1:-1, :] if d == 0 else V[:, :, :, 1:-1])
            hi, lo = C[:, 2 * d], C[:, 2 * d + 1]
            j = (lo[..., 1:] - hi[..., :-1]) if d == 0 else (lo[:, 1:] - hi[:, :-1])
            J = j[..., 1:].abs() + j[..., :-1].abs() if d == 0 else j[:, 1:].abs() + j[:, :-1].abs()
            small = D < eps
            sig = torch.where(small, 0.0, self.gk * J / torch.where(small, 1.0, D)).max(dim=0).values
            beta = self.speed(patch, d).max(dim=0).values
            expo = expo + beta * dt * sig / (self.dx, self.dy)[d]
        return torch.cat([U[:, :1], U[:, 1:] * torch.exp(-expo)], dim=1)

    def dt(self, U):
        e = self.c["k"] / 3.0 if self.c["dt_rule"] else 1.0
        rate = sum(torch.max(self.speed(U[:, 0], d)) / h ** e for d, h in zip(range(self.dim), (self.dx, self.dy)))
        return float(self.c["cfl"] / rate)

    def step(self, U, dt, t):
        L = U + dt * self.residual(U, t)
        L = L + dt * self.residual(L, t + dt)
        L = L + 0.75 * (U - L)
        L = L + dt * self.residual(L, t + 0.5 * dt)
        return self.eliminate(L + (U - L) / 3.0, dt, t + dt)


def exact(case, seed):
    c = case
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    outs, dts = [], []
    for i, (nx, ny) in enumerate(_meshes(c)):
        E = _Exact(c, nx, ny, dev)
        U = _state(c, seed + 1000 * i, dev, nx, ny).reshape(-1, 3 if c["dim"] == 2 else 2, ny, nx)
        if c["kind"] in ("adjoint", "evolve"):
            return _exact_gradient(c, E, U, seed)
        t, n = 0.0, 0
        with torch.no_grad():
            while n < c["steps"] or t < c["t_final"]:
                dt = E.dt(U)
                if c["t_final"] > 0.0 and t + dt >= c["t_final"]:
                    dt, t_next = c["t_final"] - t, c["t_final"]
                else:
                    t_next = t + dt
                U = E.step(U, dt, t)
                t, n = t_next, n + 1
                dts.append(dt)
        outs.append(U)
    if c["kind"] == "batch":
        return {"U": torch.cat([u.reshape(-1) for u in outs]), "steps": n}
    U = outs[0] if c["dim"] == 2 else outs[0][:, :, 0, :]
    if c["kind"] in ("step", "static"):
        return {"U": U, "dt": torch.tensor(dts, dtype=torch.float64, device=dev)}
    return {"U": U, "steps": n, "t": t} if c["t_final"] > 0.0 else {"U": U, "steps": n}


def _exact_gradient(c, E, U0, seed):
    from torch.utils.checkpoint import checkpoint
    dt = _fixed_dt(c)
    U0 = U0.requires_grad_(True)
    U = U0
    for _ in range(c["steps"]):
        U = checkpoint(E.step, U, dt, 0.0, use_reentrant=False)
    if c["kind"] == "evolve":
        gen = torch.Generator(device=U.device).manual_seed(int(seed))
        w = torch.randn(U.shape, dtype=torch.float64, device=U.device, generator=gen)
        (g,) = torch.autograd.grad(U, U0, w)
        return {"U": U.detach(), "grad": g}
    # integral of rho_h^2 over the cells whose centres lie in [1/4, 3/4]^2
    xc = (torch.arange(c["nx"], dtype=torch.float64, device=U.device) + 0.5) / c["nx"]
    yc = (torch.arange(c["ny"], dtype=torch.float64, device=U.device) + 0.5) / c["ny"]
    win = ((yc >= 0.25) & (yc <= 0.75))[:, None] & ((xc >= 0.25) & (xc <= 0.75))[None, :]
    r = U[0]
    J = E.dx * E.dy * torch.sum(win * (r[0] ** 2 + 12.0 * r[1] ** 2 + 12.0 * r[2] ** 2))
    (g,) = torch.autograd.grad(J, U0)
    return {"J": float(J.detach()), "grad": g}
