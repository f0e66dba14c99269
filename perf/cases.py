"""What a user of the library has it do, as measurable cases.

A case is a dict of plain values. `prepare` makes the lattice a program keeps
(mask, boundary segments, valve schedule, initial fields from a seed), `run`
is one pass through the public calls: some steps, then the fields read back
into device buffers, as a control loop, a monitor or an optimiser does
it. `exact` computes the same fields in plain FP64 PyTorch.

Kinds of lattice:
  gradient   the gradient generator with velocity inlets, outlets and valves
  channel    the straight channel between walls
  obstacles  a periodic box with random obstacles, a source patch and decay
  fluid      all fluid, periodic along x (the largest lattices, full rows)
  pressure   the gradient generator with the paper's pressure boundaries
  walls      the same with the paper's walls as well
  batch      several uneven gradient generators in one launch
  compound   the compound alone on frozen velocity fields
  adjoint    loss and gradients of the chamber misfit
"""
import math

import numpy as np
import torch

from paper_1307_4703_amd import Batch, Lattice
from paper_1307_4703_amd import workloads as W

ELEMENT = {"f64": 8, "f32": 4, "f16": 2}
FLOPS_UPDATE = 150   # one coupled update: moments, both collisions
FLOPS_COMPOUND = 35  # one compound-only update
FLOPS_ADJOINT = 45   # one adjoint update of the compound


def listed():
    return [
        # a control loop on the straight test channel: few steps between reads
        {"name": "channel_small_f64", "kind": "channel", "nx": 128, "ny": 64, "storage": "f64",
         "steps": 10, "fuse": 0, "half_period": 0},
        # a small porous box of odd size: odd step count, source and decay
        {"name": "obstacles_odd_f32", "kind": "obstacles", "nx": 333, "ny": 215, "storage": "f32",
         "steps": 37, "fuse": 0, "half_period": 0},
        # the chip at 1 um per cell, the everyday run
        {"name": "gradient_f32", "kind": "gradient", "nx": 2048, "ny": 1024, "storage": "f32",
         "steps": 256, "fuse": 5, "half_period": 2000},
        # the same as the reference precision of an error study
        {"name": "gradient_f64", "kind": "gradient", "nx": 2048, "ny": 1024, "storage": "f64",
         "steps": 128, "fuse": 5, "half_period": 2000},
        # the chip at 0.25 um per cell in the compact storage, library defaults
        {"name": "gradient_large_f16", "kind": "gradient", "nx": 8192, "ny": 4096,
         "storage": "f16", "steps": 64, "fuse": 0, "half_period": 2000},
        # the largest lattice, every node fluid, beyond every cache
        {"name": "fluid_large_f32", "kind": "fluid", "nx": 8192, "ny": 4096, "storage": "f32",
         "steps": 32, "fuse": 5, "half_period": 0},
        # a parameter study: uneven chips advanced together
        {"name": "batch_f32", "kind": "batch", "nx": 0, "ny": 0, "storage": "f32", "steps": 64,
         "fuse": 5, "half_period": 0, "members": 12},
        # long compound-only runs on the flow's frozen velocity
        {"name": "compound_f32", "kind": "compound", "nx": 2048, "ny": 1024, "storage": "f32",
         "steps": 256, "fuse": 0, "half_period": 2000},
        # the same at the paper's resolution (20-node channels, D2Q4, decay),
        # where a simulated hour is millions of steps
        {"name": "compound_paper_f32", "kind": "compound", "nx": 410, "ny": 205, "storage": "f32",
         "steps": 1200, "fuse": 0, "half_period": 500},
        # one gradient of an inverse problem
        {"name": "adjoint_f32", "kind": "adjoint", "nx": 1024, "ny": 512, "storage": "f32",
         "steps": 400, "fuse": 4, "half_period": 150},
        # the paper's pressure-driven valves
        {"name": "pressure_f32", "kind": "pressure", "nx": 2048, "ny": 1024, "storage": "f32",
         "steps": 64, "fuse": 4, "half_period": 2000},
        # the paper's full boundary set
        {"name": "walls_f32", "kind": "walls", "nx": 1024, "ny": 512, "storage": "f32",
         "steps": 40, "fuse": 0, "half_period": 2000},
    ]


def draw(rng):
    kind = rng.choice(["channel", "obstacles", "gradient", "gradient", "gradient", "fluid",
                       "fluid", "batch", "compound", "compound", "adjoint", "pressure", "walls"])

    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    c = {"kind": kind, "storage": rng.choice(["f64", "f32", "f32", "f16"]),
         "half_period": spread(20, 2000)}
    if kind == "channel":
        c |= {"nx": spread(24, 2048), "ny": spread(12, 512), "half_period": 0}
    elif kind == "obstacles":
        c |= {"nx": spread(33, 2048), "ny": spread(21, 1024), "half_period": 0}
    elif kind == "fluid":
        c |= {"nx": spread(500, 8192), "ny": spread(250, 4096), "half_period": 0}
    elif kind == "batch":
        c |= {"nx": 0, "ny": 0, "half_period": 0, "members": rng.randint(2, 15), "storage": "f32"}
    else:
        top = {"gradient": 8192, "compound": 4096, "adjoint": 1024}.get(kind, 2048)
        nx = spread(300, top)
        c |= {"nx": nx, "ny": nx // 2 + rng.randint(2, 9)}
    # the cost of a pass stays below the largest listed one's
    nodes = max(c["nx"] * c["ny"], 1) * (1 if kind in ("fluid", "obstacles", "channel") else 0.25)
    if kind == "batch":
        nodes = 0.25e6 * c["members"]
    budget = 6e8 if kind not in ("walls", "adjoint") else 1e8
    c["steps"] = spread(4, max(8, min(1500, int(budget / nodes / ELEMENT[c["storage"]] * 2))))
    if rng.random() < 0.6:
        c["steps"] = max(8, c["steps"] // 8 * 8)
    c["fuse"] = 0
    if kind in ("gradient", "fluid", "batch", "channel"):
        c["fuse"] = 5 if c["storage"] != "f16" else rng.choice([0, 4, 5])
    elif kind in ("pressure", "adjoint"):
        c["fuse"] = 4
    elif kind == "compound":
        c["steps"] = max(8, c["steps"] // 4 * 4)
    return c


# ---------------------------------------------------------------------------
# The problem a case stands for
# ---------------------------------------------------------------------------

def _wave(rng, nx, ny):
    """A smooth field in [-1, 1] of random phase: a product of two waves."""
    kx, ky = rng.uniform(1.0, 4.0, 2)
    px, py = rng.uniform(0.0, 2 * np.pi, 2)
    return np.outer(np.cos(2 * np.pi * ky * np.arange(ny) / ny + py),
                    np.cos(2 * np.pi * kx * np.arange(nx) / nx + px))


def _init(rng, nx, ny, u):
    return {"ux": u * _wave(rng, nx, ny), "uy": u * _wave(rng, nx, ny),
            "C": 0.5 + 0.45 * _wave(rng, nx, ny)}


def _workload(case):
    kind, nx, ny, st = case["kind"], case["nx"], case["ny"], case["storage"]
    if kind == "channel":
        return W.straight_channel(nx, ny, storage=st, poiseuille_init=False)
    if kind == "obstacles":
        mask = W.random_mask(nx, ny, 4703, periodic=(True, True))
        return W.Workload("obstacles", mask, tau_f=0.8, D=0.02, periodic=(True, True),
                          k_decay=1e-4, c_shift=0.5, storage=st)
    if kind == "fluid":
        wl = W.all_fluid_channel(8, 6, storage=st)
        wl.mask = np.zeros((ny, nx), np.uint8)
        return wl
    paper = kind == "compound" and nx < 600
    wl = W.gradient_generator(nx=nx, ny=ny, half_period=case["half_period"], storage=st,
                              w0=0.0 if paper else 1.0 / 3.0)
    if paper:
        wl.D, wl.k_decay = 0.00244, 3.34255e-7
    if kind in ("pressure", "walls"):
        wl.segments = [W.Segment(2, "pressure", (0, -1), rho=1.002, c_in=1.0, fix_c=True),
                       W.Segment(3, "pressure", (0, 1), rho=0.998),
                       W.Segment(4, "pressure", (0, -1), rho=1.002, c_in=0.0, fix_c=True),
                       W.Segment(5, "pressure", (0, 1), rho=0.998)]
    return wl


def _source(rng, mask):
    ny, nx = mask.shape
    R = np.zeros(mask.shape)
    y0, x0 = ny // 3, nx // 4
    h, w = min(16, ny - y0), min(24, nx - x0)
    R[y0:y0 + h, x0:x0 + w] = rng.uniform(0.0, 1e-3, (h, w))
    return np.where(mask == 0, R, 0.0)


def _problem(case, seed):
    """Workload, initial fields, source and frozen fields of one lattice."""
    rng = np.random.default_rng([seed, 4703])
    wl = _workload(case)
    ini = _init(rng, wl.nx, wl.ny, 0.02)
    if case["kind"] == "fluid":
        ini["ux"] += 0.04
    R = _source(rng, wl.mask) if case["kind"] == "obstacles" else None
    fields = None
    if case["kind"] == "compound":
        amp = 0.2 if wl.w0 == 0.0 else 0.04
        fields = [(amp * _wave(rng, wl.nx, wl.ny), amp * _wave(rng, wl.nx, wl.ny))
                  for _ in range(2)]
    return wl, ini, R, fields


def _members(case, seed):
    """The batch's chips: always the same geometries, other initial fields."""
    wls = W.batch_instances(case["members"])
    rng = np.random.default_rng([seed, 64])
    return wls, [_init(rng, w.nx, w.ny, 0.02) for w in wls]


def _lattice(case, wl, ini):
    layout = "planes" if case["kind"] == "compound" else "paired"
    lat = Lattice.from_workload(wl, init=False, layout=layout)
    if case["fuse"] and case["kind"] != "batch":
        lat.set_two_step(case["fuse"], 6)
    lat.init(**ini)
    return lat


# ---------------------------------------------------------------------------
# The measured call
# ---------------------------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "batch":
        wls, inis = _members(case, seed)
        lats = [_lattice(case, w, i) for w, i in zip(wls, inis)]
        return {"case": case, "lats": lats, "batch": Batch(lats, fuse=case["fuse"]),
                "out": [_buffers(w, 4) for w in wls]}
    wl, ini, R, fields = _problem(case, seed)
    lat = _lattice(case, wl, ini)
    state = {"case": case, "lat": lat}
    if R is not None:
        lat.set_source(R)
    if case["kind"] == "walls":
        lat.set_wall_scheme("equilibrium")
    if fields is not None:
        for slot, (ux, uy) in enumerate(fields):
            lat.set_velocity_field(slot, ux, uy)
        lat.set_phase_fields([0, 1])
    if case["kind"] == "adjoint":
        state["weight"], state["target"], state["r_box"] = W.chamber_misfit_setup(wl)
        state["weight"] = (wl.mask == 0).astype(np.float64)
    state["out"] = _buffers(wl, 1 if fields is not None else 4)
    return state


def _buffers(wl, n):
    return [torch.empty((wl.ny, wl.nx), dtype=torch.float64, device="cuda") for _ in range(n)]


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        state["batch"].step(case["steps"])
        for lat, out in zip(state["lats"], state["out"]):
            lat.read_device(*out)
        return state["out"]
    lat = state["lat"]
    if case["kind"] == "adjoint":
        r = lat.adjoint(case["steps"], state["weight"], state["target"], r_box=state["r_box"])
        lat.read_device(*state["out"])
        return {"loss": r["loss"], "d_c_in": r["d_c_in"][[0, 2]], "d_D": r["d_D"],
                "d_R": r["d_R"], "fields": state["out"]}
    if case["kind"] == "compound":
        lat.cde_step(case["steps"])
        lat.read_device(None, None, None, state["out"][0])
        return state["out"]
    lat.step(case["steps"])
    lat.read_device(*state["out"])
    return state["out"]


def work(case):
    """State read and written once, the mask read, the fields written."""
    if case["kind"] == "batch":
        wls = W.batch_instances(case["members"])
    else:
        wls = [_workload(case)]
    n, cells = sum(w.n_fluid for w in wls), sum(w.mask.size for w in wls)
    e = ELEMENT[case["storage"]]
    wide = max(4, e)
    if case["kind"] == "compound":
        return {"bytes": n * (10 * e + 4 * wide + 1) + 8 * cells,
                "flops": n * case["steps"] * FLOPS_COMPOUND}
    if case["kind"] == "adjoint":
        return {"bytes": n * (28 * e + 1) + 48 * cells,
                "flops": n * case["steps"] * (FLOPS_UPDATE + FLOPS_ADJOINT)}
    return {"bytes": n * (28 * e + 1) + 32 * cells, "flops": n * case["steps"] * FLOPS_UPDATE}


# ---------------------------------------------------------------------------
# The same in plain FP64 PyTorch
# ---------------------------------------------------------------------------

EX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
EY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)
WF = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4


class _Plain:
    """The coupled step on the list of fluid nodes: collide, gather, then the
    links that come from open segments, paper walls and pressure ghosts."""

    def __init__(self, wl, ini, R=None, walls=False):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.dev, self.wl, self.walls, self.t = dev, wl, walls, 0
        mask = torch.from_numpy(wl.mask).to(dev).to(torch.int64)
        ny, nx = mask.shape
        self.at = torch.nonzero(mask.reshape(-1) == 0).reshape(-1)
        n = self.n = self.at.numel()
        idx = torch.full((ny * nx,), -1, dtype=torch.int64, device=dev)
        idx[self.at] = torch.arange(n, device=dev)
        x, y = self.at % nx, self.at // nx
        self.x, self.y = x.double(), y.double()
        me = torch.arange(n, device=dev)
        pull, self.links, self.wall_links = [me], {}, []
        flat = mask.reshape(-1)

        def cell(xx, yy):
            inside = torch.ones_like(xx, dtype=torch.bool)
            if not wl.periodic[0]:
                inside &= (xx >= 0) & (xx < nx)
            if not wl.periodic[1]:
                inside &= (yy >= 0) & (yy < ny)
            k = (yy % ny) * nx + xx % nx
            return torch.where(inside, flat[k], 1), torch.where(inside, idx[k], -1)

        for i in range(1, 9):
            code, src = cell(x - EX[i], y - EY[i])
            pull.append(torch.where(src >= 0, i * n + src, OPP[i] * n + me))
            for s in wl.segments:
                k = torch.nonzero(code == s.id).reshape(-1)
                if k.numel():
                    self.links[i, s.id] = k
            if walls:
                k = torch.nonzero(code != 0).reshape(-1)
                partner = cell(x[k] + EX[i], y[k] + EY[i])[1]
                self.wall_links.append((i, k, code[k], partner))
        self.pull = torch.stack(pull)
        self.cs2 = (1.0 - wl.w0) / 2.0
        self.wg = [wl.w0] + [(1.0 - wl.w0) / 4.0] * 4
        self.tau_g = 0.5 + wl.D / self.cs2
        self.R = None if R is None else self.nodes(R)
        self.seg = {s.id: s for s in wl.segments}
        self.extent = {}
        for s in wl.segments:
            ys, xs = np.nonzero(wl.mask == s.id)
            c = ys if s.normal[0] else xs
            self.extent[s.id] = (c.min() - 0.5, c.max() + 0.5)
        one, zero = torch.ones(n, dtype=torch.float64, device=dev), torch.zeros(n, dtype=torch.float64, device=dev)
        rho = self.nodes(ini["rho"]) if "rho" in ini else one * wl.rho0
        ux, uy = (self.nodes(ini[q]) if q in ini else zero for q in ("ux", "uy"))
        C = self.nodes(ini["C"]) if "C" in ini else zero
        self.f = torch.stack(self.feq(rho, ux, uy))
        self.g = torch.stack(self.geq(C, ux, uy))
        self.c_in = {s.id: s.c_in for s in wl.segments}

    def nodes(self, a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(self.dev).double().reshape(-1)[self.at]

    def feq(self, rho, ux, uy, which=range(9)):
        usq = ux * ux + uy * uy
        out = []
        for i in which:
            eu = EX[i] * ux + EY[i] * uy
            out.append(rho * WF[i] * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * usq))
        return out

    def geq(self, C, ux, uy, which=range(5)):
        return [self.wg[i] * C * (1.0 + (EX[i] * ux + EY[i] * uy) / self.cs2) for i in which]

    def phase(self):
        wl = self.wl
        if not wl.schedule:
            return set(self.seg), {}, 0
        tau = (self.t - wl.t_origin) % sum(p.duration for p in wl.schedule)
        for k, p in enumerate(wl.schedule):
            if tau < p.duration:
                return set(p.open), dict(p.c_in), k
            tau -= p.duration

    def fluid_moments(self):
        f = self.f
        rho = f.sum(0)
        jx = f[1] + f[5] + f[8] - f[3] - f[6] - f[7]
        jy = f[2] + f[5] + f[6] - f[4] - f[7] - f[8]
        return rho, jx / rho, jy / rho

    def step(self, u=None, fluid=True):
        """One step; with u given, the compound alone on that velocity; with
        fluid=False the fluid's new state is left to the caller."""
        wl, f, g = self.wl, self.f, self.g
        open_, c_phase, _ = self.phase()
        rho, ux, uy = self.fluid_moments() if u is None else (None,) + tuple(u)
        C = g.sum(0)
        src = (0.0 if self.R is None else self.R) - wl.k_decay * C
        om = 1.0 / self.tau_g
        gp = torch.stack([g[i] - om * (g[i] - e) + self.wg[i] * src
                          for i, e in enumerate(self.geq(C, ux, uy))])
        gn = gp.reshape(-1)[self.pull[:5]]
        fn = fp = None
        if u is None:
            usq = ux * ux + uy * uy
            fp = torch.empty_like(f)
            for i in range(9):
                eu = EX[i] * ux + EY[i] * uy
                fp[i] = f[i] - (f[i] - rho * WF[i] * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * usq)) / wl.tau_f
            fn = fp.reshape(-1)[self.pull]
        held = {}
        for (i, sid), k in self.links.items():
            if sid not in open_:
                continue
            s, o = self.seg[sid], OPP[i]
            if s.kind == "pressure":
                held.setdefault(sid, []).append(k)
            if fn is not None:
                if s.kind == "inlet":
                    c = (self.y if s.normal[0] else self.x)[k]
                    s0, s1 = self.extent[sid]
                    us = 4.0 * s.u_max * (c - s0) * (s1 - c) / (s1 - s0) ** 2
                    eu = -(EX[o] * s.normal[0] + EY[o] * s.normal[1]) * us
                    fn[i, k] = fp[o, k] - 6.0 * WF[i] * wl.rho0 * eu
                elif s.kind == "outlet":
                    eu = (EX[i] * ux + EY[i] * uy)[k]
                    usq_k = (ux * ux + uy * uy)[k]
                    fn[i, k] = -fp[o, k] + 2.0 * WF[i] * wl.rho0 * (1.0 + 4.5 * eu * eu - 1.5 * usq_k)
                else:
                    fn[i, k] = f[i, k]
            if i < 5:
                if s.kind == "inlet":
                    gn[i, k] = -gp[o, k] + 2.0 * self.wg[i] * c_phase.get(sid, self.c_in[sid])
                elif s.kind == "outlet" or not s.fix_c:
                    gn[i, k] = gp[i, k]
                else:
                    gn[i, k] = g[i, k]
        for i, k, code, partner in self.wall_links:
            take = torch.ones_like(code, dtype=torch.bool)
            for sid in open_:
                take &= code != sid
            k, p = k[take], partner[take]
            vx, vy, Ck = -ux[k], -uy[k], C[k]
            if fn is not None:
                rs = torch.where(p >= 0, 2.0 * rho[k] - rho[p.clamp(min=0)], rho[k])
                vx, vy = vx * rho[k] / rs, vy * rho[k] / rs
                fn[i, k] = self.feq(rs, vx, vy, [i])[0]
            if i < 5:
                gn[i, k] = (self.geq(Ck, vx, vy, [i])[0]
                            + (1.0 - om) * (g[i, k] - self.geq(Ck, ux[k], uy[k], [i])[0]))
        for sid, ks in held.items():
            s, k = self.seg[sid], torch.unique(torch.cat(ks))
            if fn is not None:
                fn[:, k] = fn[:, k] * (s.rho / fn[:, k].sum(0))
            if s.fix_c:
                c = c_phase.get(sid, self.c_in[sid])
                Cn = gn[:, k].sum(0)
                rest = torch.tensor(self.wg, dtype=torch.float64, device=self.dev)[:, None] * c
                gn[:, k] = torch.where(Cn > 0, gn[:, k] * (c / Cn), rest)
        if fn is not None and fluid:
            self.f = fn
        self.g = gn
        self.t += 1
        return fn

    def grid(self, v):
        out = torch.full((self.wl.ny * self.wl.nx,), float("nan"), dtype=torch.float64, device=self.dev)
        out[self.at] = v
        return out.reshape(self.wl.ny, self.wl.nx)

    def fields(self):
        return [self.grid(v) for v in self.fluid_moments() + (self.g.sum(0),)]


def exact(case, seed):
    steps = case["steps"]
    with torch.no_grad():
        if case["kind"] == "batch":
            out = []
            for wl, ini in zip(*_members(case, seed)):
                p = _Plain(wl, ini)
                for _ in range(steps):
                    p.step()
                out.append(p.fields())
            return out
        wl, ini, R, fields = _problem(case, seed)
        p = _Plain(wl, ini, R, walls=case["kind"] == "walls")
        if case["kind"] == "adjoint":
            return _exact_adjoint(p, wl, steps)
        if fields is not None:
            fields = [(p.nodes(a), p.nodes(b)) for a, b in fields]
            for _ in range(steps):
                p.step(u=fields[p.phase()[2]])
            return [p.grid(p.g.sum(0))]
        for _ in range(steps):
            p.step()
        return p.fields()


def _exact_adjoint(p, wl, steps):
    """Reverse-mode differentiation of the compound's plain step; the fluid
    does not depend on the parameters, so it is advanced beside it."""
    _, target, (x0, y0, w, h) = W.chamber_misfit_setup(wl)
    target = p.nodes(target)
    if p.n * steps > 8e7:
        return None
    with torch.enable_grad():
        D = torch.tensor(wl.D, dtype=torch.float64, device=p.dev, requires_grad=True)
        R = torch.zeros(p.n, dtype=torch.float64, device=p.dev, requires_grad=True)
        c = {s.id: torch.tensor(v, dtype=torch.float64, device=p.dev, requires_grad=True)
             for s, v in ((s, _phase_c_in(wl, s)) for s in wl.segments if s.kind == "inlet")}
        p.tau_g = 0.5 + D / p.cs2
        p.R = R
        p.c_in = c
        for ph in wl.schedule:
            assert all(_phase_c_in(wl, p.seg[sid]) == v for sid, v in ph.c_in)
        p.phase = lambda phase=p.phase: (phase()[0], {}, 0)
        for _ in range(steps):
            p.step()
        loss = 0.5 * ((p.g.sum(0) - target) ** 2).sum()
        grads = torch.autograd.grad(loss, [D, R] + [c[s] for s in sorted(c)])
    dR = torch.nan_to_num(p.grid(grads[1]))[y0:y0 + h, x0:x0 + w]
    return {"loss": loss.detach(), "d_D": grads[0], "d_R": dR, "d_c_in": torch.stack(grads[2:]),
            "fields": [v.detach() for v in p.fields()]}


def _phase_c_in(wl, s):
    return next((v for ph in wl.schedule for sid, v in ph.c_in if sid == s.id), s.c_in)
