"""The work that a user of this library has it do, as timed passes.

Each case is one pass through the public entry points on a lattice that a user's
program has set up beforehand: time steps with the outputs a run asks for (velocity,
pressure, wall shear stress, totals, checkpoints), gradients through a run, saving
and restoring a state, and an in-situ image.  The lattices are the named workloads of
`workloads` (straight pipe, saccular aneurysm at two sizes, seeded vessel tree), a
wider tree for the largest case, and, for drawn cases, pipes, trees and periodic
channels over the whole range of sizes.

`exact` computes the same quantities in FP64 with plain torch, from the label grid and
the definitions in include/hemelb_lb.h, sharing no code with the library.
"""

import functools
import math

import numpy as np
import torch
import torch.utils.checkpoint

import workloads as wl
from paper_1906_11925_amd import LB
from paper_1906_11925_amd.autograd import LBAdjointFn
from paper_1906_11925_amd.lb import lattice_vectors, links
from workloads.camera import orbit_view, perspective_view, ramp_lut


def _steps(name, geometry, steps, lattice=15, storage="f32", bfl=False, totals=False, save=False,
           **geo):
    return dict(name=name, kind="steps", geometry=geometry, lattice=lattice, storage=storage,
                steps=steps, bfl=bfl, totals=totals, save=save, **geo)


def listed():
    return [
        # the smallest call: a tool that couples to the flow at every step
        _steps("pipe_each_step", "pipe", 1),
        # the validation pipe on the paper's lattice, stepped between two outputs
        _steps("pipe_d3q19_200", "pipe", 200, lattice=19),
        # one patient-sized aneurysm (200k sites), outputs every 100 steps
        _steps("aneurysm_half_100", "aneurysm_half", 100),
        # the same vessel with interpolated walls (the paper's wall boundary) on D3Q19
        _steps("aneurysm_half_bfl_d3q19_100", "aneurysm_half", 100, lattice=19, bfl=True),
        # a production run in 16-bit storage: steps, outputs, totals and a checkpoint
        _steps("aneurysm_f16_100", "aneurysm", 100, storage="f16", totals=True, save=True),
        # the vessel tree in FP32, outputs every 100 steps
        _steps("tree1024_100", "tree1024", 100),
        # the same tree in BF16, watched closely: outputs and totals every 10 steps
        _steps("tree1024_bf16_10", "tree1024", 10, storage="bf16", totals=True),
        # the largest: a tree of 20.8M sites (its state is many times the caches)
        _steps("tree768_wide_100", "tree", 100, r0=96, box=768, generations=6, geo_seed=3),
        # gradients of an outlet-flux and wall-shear objective with respect to the inlet
        # waveform and the Brinkman field: forward and backward with checkpoints
        dict(name="adjoint_half_checkpoints", kind="adjoint", geometry="aneurysm_half", lattice=15,
             storage="f32", steps=400, every=100, window=100),
        # the same objective on the tree from a given state, and the gradient with respect to
        # that state as well
        dict(name="adjoint_tree1024_sweep", kind="sweep", geometry="tree1024", lattice=15,
             storage="f32", steps=24, every=8, window=12),
        # saving a state and restoring it
        dict(name="tree1024_save_restore", kind="state", geometry="tree1024", lattice=15,
             storage="f32"),
        # one in-situ frame of the flow speed
        dict(name="tree1024_frame", kind="render", geometry="tree1024", lattice=15, storage="f32",
             size=1024, filter="trilinear", camera="pinhole", azimuth=35, elevation=20),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_geometry(rng, inlet, largest):
    """A pipe, tree or (without a velocity inlet) channel of up to `largest` sites."""
    n = _log_uniform(rng, 2000, largest)
    pick = rng.choice(["pipe", "tree", "tree", "named"] + ([] if inlet else ["channel"]))
    if pick == "named" and n > 300000:
        return dict(geometry=rng.choice(["aneurysm_half"] + (["aneurysm"] if largest > 1.6e6 else [])))
    if pick == "channel":
        h = max(3, int(n ** (1 / 3) * rng.uniform(0.3, 0.9)))
        x = max(3, int(n ** (1 / 3) * rng.uniform(0.3, 1.2)))
        return dict(geometry="channel", height=h, width=x, length=max(8, int(n / (h * x))))
    if pick == "tree":
        r0 = max(5.0, round((n / 23.5) ** (1 / 3), 2))
        return dict(geometry="tree", r0=r0, box=int(r0 * rng.uniform(7.0, 9.5)),
                    generations=rng.randint(3, 6), geo_seed=rng.randint(1, 1000))
    radius = max(3.3, round((n / math.pi / rng.uniform(2.0, 16.0)) ** (1 / 3), 2))
    return dict(geometry="pipe", radius=radius, length=max(8, int(n / (math.pi * radius ** 2))),
                inlet="velocity" if inlet else rng.choice(["pressure", "velocity"]))


def draw(rng):
    kind = rng.choice(["steps"] * 6 + ["adjoint", "sweep", "recorded", "state", "render"])
    lattice = rng.choice([15, 15, 19])
    storage = rng.choice(["f32", "f32", "f16", "bf16"])
    if kind == "steps":
        geo = _draw_geometry(rng, False, 1.2e7)
        bfl = geo["geometry"] not in ("tree",) and rng.random() < 0.3
        # few steps on the largest lattices, so that a pass stays below the largest listed one
        return dict(kind=kind, lattice=lattice, storage=storage, bfl=bfl,
                    steps=int(_log_uniform(rng, 1, 128)), totals=rng.random() < 0.3,
                    save=rng.random() < 0.2, **geo)
    if kind == "adjoint":
        steps = rng.randint(20, 300)
        return dict(kind=kind, lattice=lattice, storage=storage, steps=steps,
                    every=rng.randint(5, max(6, steps // 2)), window=rng.randint(5, steps),
                    **_draw_geometry(rng, True, 3e5))
    if kind in ("sweep", "recorded"):
        # recorded: the whole trajectory is kept in device memory, allocated by the pass
        steps = rng.randint(4, 40)
        every = {"every": rng.randint(2, steps)} if kind == "sweep" else {}
        return dict(kind=kind, lattice=lattice, storage=storage, steps=steps, **every,
                    window=rng.randint(1, steps),
                    **_draw_geometry(rng, True, 3e6 if kind == "sweep" else 1e5))
    if kind == "state":
        return dict(kind=kind, lattice=lattice, storage=storage, **_draw_geometry(rng, False, 1.2e7))
    return dict(kind=kind, lattice=15, storage="f32", size=rng.randint(64, 1200),
                filter=rng.choice(["nearest", "trilinear"]), camera=rng.choice(["pinhole", "orbit"]),
                azimuth=rng.randint(0, 359), elevation=rng.randint(-60, 60),
                **_draw_geometry(rng, False, 6e6))


# ----------------------------------------------------------------------------
# what the program has in hand: geometry, handle, initial state
# ----------------------------------------------------------------------------
_GEO = ("geometry", "r0", "box", "generations", "geo_seed", "radius", "length", "height", "width",
        "inlet")


def _geo_key(case):
    return tuple((k, case[k]) for k in _GEO if k in case)


@functools.lru_cache(maxsize=3)
def _geometry(key):
    c = dict(key)
    if c["geometry"] == "tree":
        mid = c["box"] / 2.0
        return wl.tree(c["box"], float(c["r0"]), (mid, mid, c["r0"] / 2.0), c["generations"],
                       seed=c["geo_seed"])
    if c["geometry"] == "channel":
        return wl.channel(H=c["height"], L=c["length"], Lx=c["width"])
    if c["geometry"] == "pipe" and "radius" in c:
        w = 2 * int(math.ceil(c["radius"])) + 3
        wave = (0.02, (0.0,), (0.01,), 4000.0) if c["inlet"] == "velocity" else None
        return wl.pipe(X=w, Y=w, Z=c["length"], r2=c["radius"] ** 2, inlet_velocity=wave)
    return wl.config_geometry(c["geometry"])


@functools.lru_cache(maxsize=3)
def _lattice_of(key, lattice, bfl):
    g = _geometry(key)
    coords, nbr = links(g.labels, g.shape, g.periodic, lattice)
    q = g.wall_fractions(lattice_vectors(lattice)) if bfl else None
    return coords, nbr, g.site_weight(), q


def _tables(lattice):
    """Lattice vectors and weights (plain definitions, rest then opposite pairs)."""
    second = ([(1, 1, 1), (1, 1, -1), (1, -1, 1), (-1, 1, 1)] if lattice == 15 else
              [(1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1), (0, 1, 1), (0, 1, -1)])
    c = [(0, 0, 0)]
    for v in [(1, 0, 0), (0, 1, 0), (0, 0, 1)] + second:
        c += [v, tuple(-a for a in v)]
    w = ([2 / 9] + [1 / 9] * 6 + [1 / 72] * 8) if lattice == 15 else ([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    return c, w


def _iolets(g, seed):
    """The geometry's iolets, the velocity inlet with a three-harmonic waveform of the seed."""
    rng = np.random.default_rng(1000 + seed)
    out = []
    for io in g.iolets:
        if io.kind == "velocity" and g.name != "couette":
            out.append(wl.Iolet("velocity", direction=io.direction, mean=io.mean * rng.uniform(0.8, 1.2),
                                cos=tuple(rng.uniform(-0.002, 0.002, 3)),
                                sin=tuple(rng.uniform(-0.004, 0.004, 3)), period=4000.0))
        else:
            out.append(io)
    return out


def _initial(case, g, coords, seed):
    """FP32 deviations of a smooth flow (|u| up to 0.02, density within 1e-3) plus
    small noise, [Q, N] on the GPU."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    cs, ws = _tables(case["lattice"])
    x = torch.from_numpy(coords).cuda()
    size = float(max(g.shape))

    def wave():
        k = rng.uniform(-6.0, 6.0, 3) / size
        ph = sum(float(k[a]) * x[:, a].to(torch.float32) for a in range(3)) + float(rng.uniform(0, 6.28))
        return torch.sin(ph)

    rho, u = 1e-3 * wave(), [0.011 * wave() for _ in range(3)]
    d = torch.empty((case["lattice"], x.shape[0]), dtype=torch.float32, device="cuda")
    d.uniform_(-2e-5, 2e-5, generator=gen)
    for i, (c, w) in enumerate(zip(cs, ws)):
        d[i] += w * (rho + 3.0 * sum(c[a] * u[a] for a in range(3) if c[a]) if i else rho)
    return d


def _alpha(n, seed):
    return np.random.default_rng(2000 + seed).uniform(0.0, 0.01, n).astype(np.float32)


def _dome(case, g, coords):
    """Sites whose wall shear enters the objective."""
    c = coords.astype(np.float64)
    if "centre" in g.info:
        m, r = np.asarray(g.info["centre"]), g.info["radius"]
        return ((c - m) ** 2).sum(axis=1) < (r + 2) ** 2
    return c[:, 2] < c[:, 2].min() + 0.25 * max(g.shape)


def _view(case, g):
    mid = [0.5 * (s - 1) for s in g.shape]
    dist = 0.9 * math.sqrt(sum(s * s for s in g.shape))
    if case["camera"] == "pinhole":
        v = perspective_view(mid, dist, case["azimuth"], case["elevation"], case["size"], case["size"])
    else:
        v = orbit_view(mid, dist, case["azimuth"], case["elevation"], case["size"], case["size"],
                       pixel=1.2 * max(g.shape) / case["size"])
    v["filter"] = case["filter"]
    return v


def _speed(n, coords, g, seed):
    """A per-site speed field of the seed, float32 [N] on the GPU."""
    rng = np.random.default_rng(3000 + seed)
    x = torch.from_numpy(coords).cuda().to(torch.float32) / float(max(g.shape))
    k = rng.uniform(4.0, 20.0, 3)
    s = sum(torch.sin(float(k[a]) * x[:, a] + float(rng.uniform(0, 6.28))) for a in range(3))
    return (0.02 + 0.006 * s).contiguous()


def prepare(case, seed):
    key = _geo_key(case)
    g = _geometry(key)
    bfl = bool(case.get("bfl"))
    coords, nbr, weight, wall_q = _lattice_of(key, case["lattice"], bfl)
    n = len(coords)
    adjoint = case["kind"] in _GRADIENTS
    lb = LB(nbr, g.tau, lattice=case["lattice"], storage=case["storage"], coords=coords,
            iolets=_iolets(g, seed), site_weight=weight, wall_q=wall_q,
            alpha=_alpha(n, seed) if adjoint else None)
    st = {"case": case, "lb": lb}
    if case["kind"] == "render":
        st["values"], st["view"], st["lut"] = _speed(n, coords, g, seed), _view(case, g), ramp_lut()
        return st
    d0 = _initial(case, g, coords, seed)
    lb.set_deviations(d0, t=0)
    if case["kind"] == "state":
        lb.step(3)
    if adjoint:
        steps = case["steps"]
        lb.set_objective(1, _Q_TARGET, _dome(case, g, coords), _LAM, (steps - case["window"], steps))
    if case["kind"] == "adjoint":
        io = lb.iolets[0]
        st["theta"] = torch.tensor([io.mean, *io.cos, *io.sin], dtype=torch.float64)
        st["alpha"] = torch.from_numpy(_alpha(n, seed))
    if case["kind"] in ("sweep", "recorded"):
        st["d0"] = d0
    return st


_GRADIENTS = ("adjoint", "sweep", "recorded")
_Q_TARGET = 0.5  # outlet flux the objective asks for
_LAM = 1.0e4     # weight of the wall-shear term


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------
def run(state):
    case, lb = state["case"], state["lb"]
    kind = case["kind"]
    if kind == "steps":
        lb.step(case["steps"])
        p, u, wss = lb.observables()
        out = {"p": p, "u": u, "wss": wss}
        if case["totals"]:
            out["totals"] = lb.totals()
        if case["save"]:
            out["state"] = lb.get_state()[0]
        return out
    if kind == "adjoint":
        theta = state["theta"].clone().requires_grad_(True)
        alpha = state["alpha"].clone().requires_grad_(True)
        J = LBAdjointFn.apply(theta, alpha, lb, 0, case["steps"], case["every"])
        dtheta, dalpha = torch.autograd.grad(J, (theta, alpha))
        return {"J": J.detach(), "dtheta": dtheta, "dalpha": dalpha}
    if kind in ("sweep", "recorded"):
        steps, every, checkpoints = case["steps"], case.get("every"), []
        lb.set_deviations(state["d0"], t=0)
        if every is None:
            lb.record(steps)
            lb.step(steps)
        else:
            for t0 in range(0, steps, every):
                k = min(every, steps - t0)
                checkpoints.append((t0, k, lb.get_state()[0]))
                lb.step(k)
        J = lb.objective_value()[0]
        lb.adjoint_begin(every or 1)
        if every is None:
            lb.adjoint_recorded()
        else:
            lb.adjoint_run(checkpoints)
        dtheta, dalpha = lb.adjoint_grads()
        dstate = lb.get_adjoint()
        lb.record_end()
        return {"J": J, "dtheta": dtheta[0], "dalpha": dalpha, "dstate": dstate}
    if kind == "state":
        saved, t = lb.get_state()
        lb.set_state(saved, t)
        return {"state": saved, "deviations": lb.get_deviations()}
    return {"image": lb.render(state["values"], state["view"], state["lut"], scale=20.0, offset=0.0)}


def work(case):
    """Bytes and operations of one pass, each population read and written once a step."""
    n = len(_lattice_of(_geo_key(case), case["lattice"], bool(case.get("bfl")))[0])
    q = case["lattice"]
    pop = q * (4 if case["storage"] == "f32" else 2)
    flop = 8 * q + 30  # moments, equilibrium and relaxation of one site
    if case["kind"] == "steps":
        b = n * (2.0 * pop * case["steps"] + pop + 20)
        if case["totals"]:
            b += n * pop
        if case["save"]:
            b += 2 * n * pop
        return {"bytes": b, "flops": float(n * flop * (case["steps"] + 1))}
    if case["kind"] in _GRADIENTS:
        s = case["steps"]
        forward = n * 2.0 * pop * s * (1 if case["kind"] == "recorded" else 2)
        # reverse: adjoint populations in and out, the taped state, the Brinkman field and
        # its FP64 gradient
        reverse = n * s * (2.0 * 4 * q + pop + 4 + 16)
        return {"bytes": forward + reverse, "flops": float(n * s * flop * 4)}
    if case["kind"] == "state":
        return {"bytes": n * (5.0 * pop + 4 * q), "flops": 0.0}
    rays = case["size"] ** 2
    # the field once, the image once; a ray crosses about a tenth of the box's extent in fluid
    return {"bytes": 4.0 * n + 16.0 * rays, "flops": float(rays * 40 * 30)}


# ----------------------------------------------------------------------------
# FP64 values of the same outputs
# ----------------------------------------------------------------------------
def _site_grid(g):
    """(int32 grid of site indices over the padded box, -1 elsewhere; coords [N, 3])."""
    lab = torch.from_numpy(g.labels).cuda()
    X, Y, Z = g.shape
    fluid = torch.zeros_like(lab, dtype=torch.bool)
    fluid[1:X + 1, 1:Y + 1, 1:Z + 1] = lab[1:X + 1, 1:Y + 1, 1:Z + 1] == 1
    flat = fluid.view(-1).nonzero().view(-1)
    grid = torch.full(lab.shape, -1, dtype=torch.int32, device="cuda")
    grid.view(-1)[flat] = torch.arange(len(flat), dtype=torch.int32, device="cuda")
    YZ, Zp = lab.shape[1] * lab.shape[2], lab.shape[2]
    xyz = torch.stack([flat // YZ, (flat // Zp) % lab.shape[1], flat % Zp], dim=1) - 1
    return lab, grid, xyz


class _Exact:
    """The time step of include/hemelb_lb.h in FP64, differentiable."""

    def __init__(self, case, g, iolets, weight, alpha=None, wall_q=None):
        self.cs, ws = _tables(case["lattice"])
        self.q, self.omega = len(self.cs), 1.0 / g.tau
        self.w = torch.tensor(ws, dtype=torch.float64, device="cuda")
        self.iolets, self.alpha = iolets, alpha
        lab, grid, xyz = _site_grid(g)
        n = self.n = len(xyz)
        here = torch.arange(n, device="cuda")
        idx = torch.empty((self.q, n), dtype=torch.int64, device="cuda")
        idx[0] = here
        self.links = []   # (iolet, direction, sites)
        self.walls = []   # (direction, sites)
        self.normal = torch.zeros((3, n), dtype=torch.float64, device="cuda")
        self.fluid = {}
        for i in range(1, self.q):
            y = xyz - torch.tensor(self.cs[i], device="cuda")
            for a in range(3):
                if g.periodic[a]:
                    y[:, a] %= g.shape[a]
            at = ((y[:, 0] + 1) * lab.shape[1] + y[:, 1] + 1) * lab.shape[2] + y[:, 2] + 1
            src, kind = grid.view(-1)[at].long(), lab.view(-1)[at]
            idx[i] = torch.where(src >= 0, i * n + src, self.opp(i) * n + here)
            wall = ((src < 0) & (kind == 0)).nonzero().view(-1)
            self.walls.append((i, wall))
            for a in range(3):
                self.normal[a, wall] += self.cs[i][a]
            for k in range(len(iolets)):
                s = ((src < 0) & (kind == 2 + k)).nonzero().view(-1)
                if len(s):
                    self.links.append((k, i, s))
            if wall_q is not None:
                self.fluid[i] = src >= 0
        del grid, lab
        self.idx = idx.view(-1)
        norm = self.normal.norm(dim=0)
        self.has = norm > 0
        self.normal = torch.where(self.has, self.normal / norm.clamp(min=1e-300), self.normal)
        self.weight = torch.from_numpy(weight).cuda()
        self.wall_q = None
        if wall_q is not None:
            q = torch.from_numpy(np.nan_to_num(wall_q, nan=0.5).astype(np.float32)).cuda().double()
            self.wall_q = (q * 32768.0).round().clamp(1, 32768) / 32768.0

    @staticmethod
    def opp(i):
        return 0 if i == 0 else (i + 1 if i % 2 else i - 1)

    def moments(self, f):
        m = [sum(f[i] * c[a] for i, c in enumerate(self.cs) if c[a]) for a in range(3)]
        return f.sum(dim=0), m

    def feq(self, rho, u):
        usq = 1.5 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2])
        rows = []
        for i, c in enumerate(self.cs):
            cu = sum((u[a] * c[a] for a in range(3) if c[a]), torch.zeros_like(rho))
            rows.append(self.w[i] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - usq))
        return torch.stack(rows)

    def value(self, k, t, theta):
        io = self.iolets[k]
        th = theta if theta is not None and io.kind == "velocity" else [io.mean, *io.cos, *io.sin]
        h = (len(th) - 1) // 2
        v = th[0]
        for j in range(h):
            ph = 2.0 * math.pi * (j + 1) * t / io.period
            v = v + th[1 + j] * math.cos(ph) + th[1 + h + j] * math.sin(ph)
        return v

    def stream(self, A, t, theta=None):
        n = self.n
        f = A.reshape(-1).index_select(0, self.idx)
        if self.wall_q is not None:
            f0 = f.view(self.q, n)
            g = f0.clone()
            for i, s in self.walls:
                o, q = self.opp(i), self.wall_q[s, i]
                near = torch.where(self.fluid[o][s], 2 * q * A[o, s] + (1 - 2 * q) * f0[o, s], A[o, s])
                far = A[o, s] / (2 * q) + (2 * q - 1) / (2 * q) * A[i, s]
                g[i, s] = torch.where(q < 0.5, near, far)
            f = g.view(-1)
        pos, val = [], []
        for k, i, s in self.links:
            io = self.iolets[k]
            if io.kind == "pressure":
                rho, m = self.moments(A[:, s])
                u = [x / rho for x in m]
                cu = sum(u[a] * self.cs[i][a] for a in range(3) if self.cs[i][a])
                usq = sum(x * x for x in u)
                v = self.w[i] * self.value(k, t, theta) * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * usq)
            else:
                ce = sum(self.cs[i][a] * io.direction[a] for a in range(3))
                v = A[self.opp(i), s] + 6 * self.w[i] * ce * self.value(k, t, theta) * self.weight[s]
            pos.append(i * n + s)
            val.append(v)
        if pos:
            f = f.index_copy(0, torch.cat(pos), torch.cat(val))
        return f.view(self.q, n)

    def step(self, A, t, theta=None):
        f = self.stream(A, t, theta)
        rho, m = self.moments(f)
        damp = 1.0 if self.alpha is None else 1.0 - self.alpha
        return f - self.omega * (f - self.feq(rho, [damp * x / rho for x in m])), f

    def shear(self, f, s=None):
        """Wall shear stress at sites s (all: None)."""
        nrm = self.normal if s is None else self.normal[:, s]
        rho, m = self.moments(f)
        e = f - self.feq(rho, [x / rho for x in m])
        k = -(1.0 - 0.5 * self.omega)
        tr = [k * sum(self.cs[i][a] * self.cs[i][b] * e[i] * nrm[b] for i in range(self.q)
                      for b in range(3) if self.cs[i][a] and self.cs[i][b]) for a in range(3)]
        nsn = sum(tr[a] * nrm[a] for a in range(3))
        t2 = sum((tr[a] - nsn * nrm[a]) ** 2 for a in range(3))
        ok = (self.has if s is None else self.has[s]) & (t2 > 0)
        return torch.where(ok, torch.where(ok, t2, torch.ones_like(t2)).sqrt(), torch.zeros_like(t2))

    def flux(self, A, f, outlet):
        return sum((A[self.opp(i), s] - f[i, s]).sum() for k, i, s in self.links if k == outlet)


def _exact_gradients(case, g, E, A, theta, dome, want_state):
    steps, window = case["steps"], case["window"]
    dome = torch.from_numpy(dome).cuda() & E.has
    sites = dome.nonzero().view(-1)

    def one(A, t, theta, alpha):
        E.alpha = alpha
        A1, f = E.step(A, t, theta)
        if t < steps - window:
            return A1, A1.new_zeros(())
        Q = E.flux(A, f, 1)
        w = E.shear(f[:, sites], sites).mean() if len(sites) else A1.new_zeros(())
        return A1, (Q - _Q_TARGET) ** 2 + _LAM * w / window

    alpha = E.alpha.requires_grad_(True)
    A = A.requires_grad_(want_state)
    J, B = 0.0, A
    for t in range(steps):
        B, j = torch.utils.checkpoint.checkpoint(one, B, t, theta, alpha, use_reentrant=False)
        J = J + j
    grads = torch.autograd.grad(J, (theta, alpha) + ((A,) if want_state else ()))
    return J.detach().cpu(), [x.detach() for x in grads]


def _exact_image(case, g, seed):
    """The ray-marched image of include/hemelb_lb.h, all rays side by side."""
    lab, grid, xyz = _site_grid(g)
    vals = _speed(len(xyz), xyz.to(torch.int32).cpu().numpy(), g, seed)
    v, n = _view(case, g), case["size"]
    dims = torch.tensor(g.shape, device="cuda")
    fix = 1 << 20
    jj, ii = torch.meshgrid(torch.arange(n, device="cuda"), torch.arange(n, device="cuda"), indexing="ij")
    ii, jj = ii.reshape(-1), jj.reshape(-1)

    def vec(name):
        return torch.tensor(v.get(name, (0, 0, 0)), dtype=torch.int64, device="cuda")

    P0 = vec("origin") + ii[:, None] * vec("right") + jj[:, None] * vec("up")
    D = vec("dir") + ii[:, None] * vec("dir_right") + jj[:, None] * vec("dir_up")
    lut = torch.from_numpy(ramp_lut()).cuda().double()
    C = torch.zeros((n * n, 4), dtype=torch.float64, device="cuda")

    def site(x):
        ok = ((x >= 0) & (x < dims)).all(dim=1)
        y = torch.where(ok[:, None], x, torch.zeros_like(x)) + 1
        s = grid.view(-1)[(y[:, 0] * lab.shape[1] + y[:, 1]) * lab.shape[2] + y[:, 2]].long()
        return torch.where(ok, s, torch.full_like(s, -1))

    for k in range(v["steps"]):
        P = P0 + k * D
        near = ((P >= -2 * fix) & (P < (dims + 2) * fix)).all(dim=1).nonzero().view(-1)
        if not len(near):
            continue
        P = P[near]
        if v["filter"] == "nearest":
            s = site((P + fix // 2) >> 20)
            hit, val = s >= 0, vals[s.clamp(min=0)].double()
        else:
            b = P >> 20
            fr = (P - b * fix) >> 12
            val = torch.zeros(len(near), dtype=torch.float64, device="cuda")
            hit = torch.zeros(len(near), dtype=torch.bool, device="cuda")
            for c in range(8):
                o = torch.tensor([c & 1, c >> 1 & 1, c >> 2 & 1], device="cuda")
                W = torch.where(o.bool(), fr, 256 - fr).prod(dim=1)
                s = site(b + o)
                ok = (s >= 0) & (W > 0)
                val += torch.where(ok, W.double() * vals[s.clamp(min=0)].double(), 0.0)
                hit |= ok
            val = val / 2.0 ** 24
        t = (val.float() - 0.0) * 20.0  # the table entry is chosen in FP32 by definition
        e = (t * 256.0).floor().clamp(0, 255).long()
        near, rgba = near[hit], lut[e[hit]]
        w = (1.0 - C[near, 3]) * rgba[:, 3]
        C[near] += torch.cat([w[:, None] * rgba[:, :3], w[:, None]], dim=1)
    return {"image": C.view(n, n, 4)}


def exact(case, seed):
    key = _geo_key(case)
    g = _geometry(key)
    if case["kind"] == "render":
        # whole images of many thousand samples a ray take too long here
        return _exact_image(case, g, seed) if case["size"] ** 2 * max(g.shape) <= 2 ** 30 else None
    bfl = bool(case.get("bfl"))
    wall_q = g.wall_fractions(np.array(_tables(case["lattice"])[0])) if bfl else None
    lab = torch.from_numpy(g.labels[1:-1, 1:-1, 1:-1] == 1)
    coords = lab.nonzero().to(torch.int32).numpy()
    n = len(coords)
    q, adjoint = case["lattice"], case["kind"] in _GRADIENTS
    work_size = n * q * (case.get("steps", 3) * (8 if adjoint else 1))
    if work_size > 4e10:
        return None
    alpha = torch.from_numpy(_alpha(n, seed)).cuda().double() if adjoint else None
    E = _Exact(case, g, _iolets(g, seed), g.site_weight(), alpha, wall_q)
    w = E.w[:, None]
    if case["kind"] == "adjoint":
        A = w.repeat(1, n)
    else:
        A = _initial(case, g, coords, seed).double() + w
    if adjoint:
        io = E.iolets[0]
        theta = torch.tensor([io.mean, *io.cos, *io.sin], dtype=torch.float64,
                             device="cuda").requires_grad_(True)
        J, gr = _exact_gradients(case, g, E, A, theta, _dome(case, g, coords), case["kind"] != "adjoint")
        out = {"J": J, "dtheta": gr[0], "dalpha": gr[1]}
        if case["kind"] != "adjoint":
            out["dstate"] = gr[2]
        return out
    f = None
    for t in range(case.get("steps", 3)):
        A, f = E.step(A, t)
    if case["kind"] == "state":
        return {"state": _stored(case, A - w), "deviations": A - w}
    rho, m = E.moments(f)
    out = {"p": (rho - 1.0) / 3.0, "u": torch.stack([x / rho for x in m], dim=1), "wss": E.shear(f)}
    if case["totals"]:
        out["totals"] = torch.stack([A.sum(), *(x.sum() for x in E.moments(A)[1])])
    if case["save"]:
        out["state"] = _stored(case, A - w)
    return out


def _stored(case, d):
    """Deviations in the units of a saved state: 16-bit storage multiplies each
    direction by the power of two nearest to 1 / w_i from below (rest 4 for D3Q15)."""
    if case["storage"] == "f32":
        return d
    scale = [4.0] + [8.0] * 6 + [64.0] * 8 if case["lattice"] == 15 else [4.0] + [16.0] * 6 + [32.0] * 12
    return d * torch.tensor(scale, dtype=torch.float64, device="cuda")[:, None]
