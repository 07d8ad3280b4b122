"""The work that a user of this library has it do, as measurable cases.

A case is one pass of a user's program through the public binding
(`paper_2606_31707_amd.hlbm`, `.autograd`): a simulation advanced by a block of
steps, a mean-flow window, an adjoint solve with its gradient, a whole gradient
evaluation, or a tick of the packed serving launches.  The geometries are this
repository's own (`inputs.py`, the serving mix, the roofline grid): a porous
cylinder in a channel with a velocity inlet and a pressure outlet.

`exact` gives what a pass returns in plain torch float64: the collisions, the
streaming and the objectives written from their definitions, the adjoint by
automatic differentiation of the per-cell collision and of the streaming.
"""
from __future__ import annotations

import math

import torch

from paper_2606_31707_amd import autograd as A
from paper_2606_31707_amd import hlbm as H

DEV = "cuda"
PRECISIONS = {"fp64": H.FP64, "fp32": H.FP32, "fp16s": H.FP16S}


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------

def _case(name=None, **kw):
    c = dict(kind="primal", dim=2, precision="fp32", nx=256, ny=128, nz=1, walls=True, u_max=0.04, re=100.0,
             cs=0.0, hrr=False, d_frac=0.25, x_frac=0.25, objective="ffa", steps=0, window=0, adjoint=0,
             tol=0.0, check=100, tau_adj=0.0, diff=False, probe=False, members=1, nx_last=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The small validation channel (220 x 41, Re 20): a block of steps with the steady
        # criterion checked every 100 of them.  The smallest calls: launches and latency.
        _case("channel_220x41_fp64_steady", precision="fp64", nx=220, ny=41, u_max=0.03, re=20.0, d_frac=10 / 41,
              x_frac=40 / 220, steps=400, tol=1e-12),
        # One evaluation of the differentiable objective (forward and backward of the
        # torch.autograd.Function) on the 400 x 160 Re 40 optimisation lattice.
        _case("objective_400x160_fp64", kind="autograd", precision="fp64", nx=400, ny=160, u_max=0.03, re=40.0,
              x_frac=0.4, steps=400, adjoint=400),
        # The vortex-street channel (1100 x 410, Re 100): a block of the long spin-up, with
        # the velocity probe from which the shedding period is read.
        _case("vortex_1100x410_fp64_steps", precision="fp64", nx=1100, ny=410, d_frac=40 / 410, x_frac=160 / 1100,
              steps=400, probe=True),
        # The same channel's mean-flow dissipation gradient: window over a large region, then
        # the adjoint at tau_adj 0.6 and the gradient.  An odd window length.
        _case("vortex_1100x410_fp32_gradient", kind="query", nx=1100, ny=410, d_frac=40 / 410, x_frac=160 / 1100,
              objective="diss", window=201, adjoint=200, tau_adj=0.6),
        # The large 2D grid (33.5 M cells, larger than every cache): the streaming sweep.
        _case("grid_8192x4096_fp32_steps", nx=8192, ny=4096, d_frac=1 / 16, x_frac=1 / 8, steps=60),
        # The same grid with 16-bit storage: window with a drag plane, adjoint, gradient.
        _case("grid_8192x4096_fp16s_gradient", kind="query", precision="fp16s", nx=8192, ny=4096, d_frac=1 / 16,
              x_frac=1 / 8, window=32, adjoint=32),
        # One serving tick: a dozen small channels in different phases (primal, window,
        # adjoint) advanced 256 steps by packed launches.
        _case("serving_packed_fp32", kind="group", members=12, nx=128, nx_last=512, ny=0, u_max=0.05, re=60.0,
              steps=256),
        # The serving mix's 1024 x 512 query, least viscous (closure on, frozen in the adjoint).
        _case("serving_1024x512_fp32_query", kind="query", nx=1024, ny=512, u_max=0.05, re=500.0, cs=0.1, steps=64,
              window=64, adjoint=128),
        # A 3D gradient with the recursive regularised collision, 16-bit storage, the closure
        # differentiated (mean populations tracked), on the serving mix's 192 x 96 x 64.
        _case("hrr_192x96x64_fp16s_gradient", kind="query", dim=3, precision="fp16s", nx=192, ny=96, nz=64,
              u_max=0.05, re=400.0, cs=0.1, hrr=True, diff=True, objective="diss", window=32, adjoint=32),
        # The steady 3D validation lattice (756 x 168 x 84, Re 40, periodic sides) in FP64.
        _case("porous_756x168x84_fp64_steps", dim=3, precision="fp64", nx=756, ny=168, nz=84, walls=False,
              u_max=0.0317, re=40.0, d_frac=1 / 8, x_frac=1 / 3, steps=24),
        # The 3D LES lattice (37.7 M cells, Re 3900): a block of its mean-flow window with the
        # drag plane, and ...
        _case("les_768x384x128_fp32_window", kind="window", dim=3, nx=768, ny=384, nz=128, walls=False, re=3900.0,
              cs=0.1, d_frac=1 / 8, steps=8, window=24),
        # ... a block of its frozen-turbulence adjoint at tau_adj 0.6, with the gradient.
        _case("les_768x384x128_fp32_adjoint", kind="adjoint", dim=3, nx=768, ny=384, nz=128, walls=False, re=3900.0,
              cs=0.1, d_frac=1 / 8, window=4, adjoint=24, tau_adj=0.6),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    """One more case of the same ranges: 2D channels from 96 x 40 to 8192 x 4096, 3D ones from
    64 x 48 x 16 to 768 x 384 x 128, any precision form, odd sizes and step counts among them."""
    kind = rng.choice(["primal", "primal", "window", "query", "query", "adjoint", "autograd", "group"])
    prec = rng.choice(["fp64", "fp32", "fp32", "fp16s"])
    if kind == "group":
        nx = _log(rng, 96, 256)
        return _case(kind=kind, precision=prec, members=rng.randint(2, 12), nx=nx, nx_last=nx + rng.randint(0, 256),
                     ny=0, u_max=0.05, re=rng.uniform(20, 200), steps=rng.randint(16, 256))
    dim = 2 if kind == "autograd" else rng.choice([2, 2, 2, 3])
    if dim == 2:
        nx = _log(rng, 96, 8192)
        ny, nz = max(40, int(nx * rng.uniform(0.25, 0.5))), 1
        walls = rng.random() < 0.8
    else:
        nx = _log(rng, 64, 768)
        ny = max(16, int(nx * rng.uniform(0.35, 0.5)))
        nz = max(8, int(nx * rng.uniform(0.08, 1 / 6)))
        walls = rng.random() < 0.4
    big = nx * ny * nz * (9 if dim == 2 else 19) > 50_000_000
    a, b = (8, 20) if big else (16, 200)
    cs = rng.choice([0.0, 0.1])
    hrr = rng.random() < 0.25
    diff = cs > 0 and not big and rng.random() < 0.3
    return _case(kind=kind, dim=dim, precision=prec, nx=nx, ny=ny, nz=nz, walls=walls,
                 u_max=rng.uniform(0.02, 0.05), re=rng.uniform(20, 200), cs=cs, hrr=hrr,
                 d_frac=rng.uniform(0.1, 0.25), x_frac=rng.uniform(0.2, 0.4),
                 objective=rng.choice(["ffa", "diss"]),
                 steps=rng.randint(a, b), window=rng.randint(a, b), adjoint=2 * rng.randint(a // 2, b // 2),
                 tau_adj=rng.choice([0.0, 0.6]), diff=diff, probe=rng.random() < 0.3)


# --------------------------------------------------------------------------
# what a program holds before the call
# --------------------------------------------------------------------------

class _Setup:
    """Sizes, parameters and seeded fields of one channel."""

    def __init__(self, case, seed):
        c = self.case = case
        self.dim = c["dim"]
        self.nx, self.ny, self.nz = c["nx"], c["ny"], c["nz"]
        self.n = self.nx * self.ny * self.nz
        self.q = 9 if self.dim == 2 else 19
        self.D = c["d_frac"] * self.ny
        self.xc, self.yc = c["x_frac"] * self.nx, (self.ny - 1) / 2.0
        self.u_max, self.walls = c["u_max"], c["walls"]
        u_mean = 2.0 / 3.0 * self.u_max if self.walls else self.u_max
        # without the closure the drawn Reynolds numbers stop where the relaxation time gets
        # too small to be stable
        self.tau = max(3.0 * u_mean * self.D / c["re"] + 0.5, 0.5014 if c["cs"] > 0 else 0.53)
        self.tau_adj = c["tau_adj"] if c["tau_adj"] > 0 else self.tau
        self.cs, self.hrr, self.diff = c["cs"], c["hrr"], c["diff"]
        self.track = bool(self.diff or self.hrr)
        hi = (self.ny - 1, self.nz - 1)
        if c["objective"] == "ffa":  # drag plane downstream of the cylinder
            x = min(self.nx - 2, int(self.xc + 4 * self.D))
            self.lo, self.hi = (x, 0, 0), (x,) + hi
        else:  # dissipation box around it
            self.lo = (max(1, int(self.xc - 2 * self.D)), 0, 0)
            self.hi = (min(self.nx - 2, int(self.xc + 6 * self.D)),) + hi
        self.kind = H.OBJ_FFA if c["objective"] == "ffa" else H.OBJ_DISS
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(int(seed))

    def fields(self):
        """Porosity noise [n] in the cylinder's box and initial velocity [3, n]: the inflow
        continued into the domain plus one per cent of noise."""
        noise = 0.05 * torch.rand(self.n, generator=self.gen, device=DEV, dtype=torch.float64)
        u = 0.02 * self.u_max * (torch.rand(3, self.n, generator=self.gen, device=DEV, dtype=torch.float64) - 0.5)
        u.view(3, self.nz, self.ny, self.nx)[0] += self.inflow()[None, :, None]
        if self.dim == 2:
            u[2].zero_()
        return noise, u.view(-1)

    def inflow(self):
        y = torch.arange(self.ny, device=DEV, dtype=torch.float64)
        if not self.walls:
            return torch.full_like(y, self.u_max)
        return 4.0 * self.u_max * (y + 0.5) * (self.ny - 0.5 - y) / (self.ny * self.ny)

    def lattice(self, stream=None):
        return H.Lattice(stencil=H.D2Q9 if self.dim == 2 else H.D3Q19, precision=PRECISIONS[self.case["precision"]],
                         nx=self.nx, ny=self.ny, nz=self.nz, tau=self.tau, cs=self.cs,
                         bc_y=H.BC_WALLS if self.walls else H.BC_PERIODIC, u_in=self.u_max,
                         inlet_profile=H.INLET_PARABOLIC if self.walls else H.INLET_UNIFORM,
                         track_mean_populations=self.track, collision=H.COLL_HRR if self.hrr else H.COLL_BGK,
                         stream=stream)

    def build(self, stream=None):
        lat = self.lattice(stream)
        noise, u = self.fields()
        torch.cuda.current_stream().synchronize()
        lat.build_cylinder(self.xc, self.yc, self.D, noise, H.NOISE_BOX, 2.0 * self.D)
        lat.init_equilibrium(1.0, u)
        lat.set_objective(self.kind, self.lo, self.hi, u0=self.u_max)
        return lat

    def porosity(self, noise):
        """The same field in float64 (solid fraction: a cosine ramp over two cells, plus the
        noise inside the box)."""
        x = torch.arange(self.nx, device=DEV, dtype=torch.float64) - self.xc
        y = torch.arange(self.ny, device=DEV, dtype=torch.float64) - self.yc
        r = torch.sqrt(x[None, :] ** 2 + y[:, None] ** 2)
        R = 0.5 * self.D
        chi = 0.5 * (1.0 + torch.cos(math.pi * (r - R + 1.0) * 0.5))
        chi = torch.where(r <= R - 1, torch.ones_like(chi), torch.where(r >= R + 1, torch.zeros_like(chi), chi))
        box = (x[None, :].abs() <= 2 * self.D) & (y[:, None].abs() <= 2 * self.D)
        chi = chi.expand(self.nz, self.ny, self.nx)
        chi = torch.where(box, (chi + noise.view(self.nz, self.ny, self.nx)).clamp(0.0, 1.0), chi)
        return 1.0 - chi


def _member(case, k):
    """Member k of a serving tick: sizes spread over [nx, nx_last], phases in turn."""
    m = max(1, case["members"] - 1)
    nx = case["nx"] + (case["nx_last"] - case["nx"]) * k // m
    return dict(case, nx=nx, ny=nx // 2, objective=("ffa", "diss")[k % 2]), (0, 1, 2)[k % 3]


def _buffers(s, names):
    size = {"populations": s.q * s.n, "rho": s.n, "u": 3 * s.n, "mean_rho": s.n, "mean_u": 3 * s.n, "mean_tau": s.n,
            "gradient": s.n}
    return {k: torch.empty(size[k], dtype=torch.float64, device=DEV) for k in names}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "group":
        stream = torch.cuda.Stream()
        group, lats, modes, outs = H.Group(stream.cuda_stream), [], [], []
        for k in range(case["members"]):
            c, mode = _member(case, k)
            s = _Setup(c, seed * 64 + k)
            lat = s.build(stream.cuda_stream)
            if mode == H.GROUP_ADJOINT:
                lat.solve_adjoint(H.SOURCE_STEADY, turb=H.TURB_FROZEN, max_iters=0)
            lats.append(lat)
            modes.append(mode)
            outs.append(_buffers(s, (("populations",), ("populations", "mean_rho", "mean_u"), ("gradient",))[mode]))
        return {"case": case, "group": group, "lats": lats, "modes": modes, "outs": outs, "stream": stream}
    s = _Setup(case, seed)
    if kind == "autograd":
        noise, u = s.fields()
        d = s.porosity(noise).reshape(-1).clone()
        lat = A.make_lattice(stencil=H.D2Q9 if s.dim == 2 else H.D3Q19, precision=PRECISIONS[case["precision"]],
                             nx=s.nx, ny=s.ny, nz=s.nz, tau=s.tau, cs=s.cs, u_in=s.u_max,
                             bc_y=H.BC_WALLS if s.walls else H.BC_PERIODIC,
                             inlet_profile=H.INLET_PARABOLIC if s.walls else H.INLET_UNIFORM,
                             track_mean_populations=s.track, collision=H.COLL_HRR if s.hrr else H.COLL_BGK)
        lat.set_objective(s.kind, s.lo, s.hi, u0=s.u_max)
        # an optimisation loop starts each primal from the state it has
        lat.set_porosity(d)
        lat.init_equilibrium(1.0, u)
        start = lat.populations(out=torch.empty(s.q * s.n, dtype=torch.float64, device=DEV))
        plan = A.Plan(primal_steps=case["steps"], adjoint_iters=case["adjoint"], tau_adj=case["tau_adj"],
                      initial_populations=start, turb=H.TURB_DIFFERENTIATED if s.diff else H.TURB_FROZEN)
        return {"case": case, "d": d.requires_grad_(True), "lat": lat, "plan": plan}
    lat = s.build()
    st = {"case": case, "lat": lat, "turb": H.TURB_DIFFERENTIATED if s.diff else H.TURB_FROZEN}
    if kind == "primal":
        if case["probe"]:
            lat.set_probe(min(s.nx - 2, int(s.xc + 2 * s.D)), int(s.yc), s.nz // 2)
        st["out"] = _buffers(s, ("populations",))
    elif kind == "window":
        lat.run_primal(case["steps"])
        st["out"] = _buffers(s, ("rho", "u", "mean_rho", "mean_u") + (("mean_tau",) if s.cs > 0 else ()))
    elif kind == "adjoint":
        lat.run_primal(case["window"], accumulate=True)
        st["out"] = _buffers(s, ("gradient",))
    else:  # query: every evaluation starts from the state in hand
        st["start"] = lat.populations(out=torch.empty(s.q * s.n, dtype=torch.float64, device=DEV))
        st["out"] = _buffers(s, ("populations", "mean_u", "gradient"))
    lat.synchronize()
    return st


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

_FIELDS = {"rho": H.FIELD_RHO, "u": H.FIELD_U, "mean_rho": H.FIELD_MEAN_RHO, "mean_u": H.FIELD_MEAN_U,
           "mean_tau": H.FIELD_MEAN_TAU}


def _read(lat, out):
    for k, t in out.items():
        if k == "populations":
            lat.populations(out=t)
        elif k == "gradient":
            lat.gradient(out=t)
        else:
            lat.field(_FIELDS[k], out=t)
    return dict(out)


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "group":
        group = state["group"]
        group.set(state["lats"], state["modes"])
        group.step(c["steps"])
        group.synchronize()
        return [_read(lat, out) for lat, out in zip(state["lats"], state["outs"])]
    lat = state["lat"]
    if kind == "autograd":
        d = state["d"]
        d.grad = None
        J = A.objective(d, lat, state["plan"])
        J.backward()
        return {"J": J.detach(), "gradient": d.grad}
    if kind == "primal":
        lat.run_primal(c["steps"], steady_tol=c["tol"], check_every=c["check"])
        r = _read(lat, state["out"])
        r["J"] = lat.objective()
        if c["probe"]:
            r["probe"] = lat.probe()[-c["steps"]:]
        return r
    if kind == "window":
        lat.window_reset()
        lat.run_primal(c["window"], accumulate=True)
        r = _read(lat, state["out"])
        r["J"] = lat.window_objective()
        return r
    if kind == "query":
        lat.set_populations(state["start"])
        lat.window_reset()
        if c["steps"]:
            lat.run_primal(c["steps"])
        lat.run_primal(c["window"], accumulate=True)
    lat.solve_adjoint(H.SOURCE_MEAN, tau_adj=c["tau_adj"], turb=state["turb"], max_iters=c["adjoint"])
    r = _read(lat, state["out"])
    r["J"] = lat.window_objective()
    return r


def work(case):
    """Bytes: the state and the porosity read once, what the pass returns or leaves behind
    written once, for the whole block of steps.  Operations: per cell and step, counted on the
    update's formulas (pairs of opposite directions, no zero coefficients)."""
    if case["kind"] == "group":
        w = {"bytes": 0.0, "flops": 0.0}
        for k in range(case["members"]):
            c, mode = _member(case, k)
            one = work(dict(c, kind=("primal", "window", "adjoint")[mode], window=c["steps"], adjoint=c["steps"]))
            w = {key: w[key] + one[key] for key in w}
        return w
    q, dim = (9, 2) if case["dim"] == 2 else (19, 3)
    n = case["nx"] * case["ny"] * case["nz"]
    s = {"fp64": 8, "fp32": 4, "fp16s": 2}[case["precision"]]
    a = 8 if case["precision"] == "fp64" else 4
    step = (110 if dim == 2 else 250) + (50 if case["cs"] > 0 else 0) + ((100 if dim == 2 else 250) if case["hrr"] else 0)
    adj = (120 if dim == 2 else 260) + ((150 if dim == 2 else 400) if case["hrr"] else 0) + (60 if case["diff"] else 0)
    kind = case["kind"]
    primal = {"primal": case["steps"], "window": case["window"], "adjoint": 0, "autograd": case["steps"],
              "query": case["steps"] + case["window"]}[kind]
    window = case["window"] if kind in ("window", "query") else 0
    adjoint = case["adjoint"] if kind in ("adjoint", "query", "autograd") else 0
    flops = n * (primal * step + window * (dim + 2) + adjoint * adj)
    if kind == "adjoint":
        bytes_ = n * (a + 8 * (1 + dim))  # porosity and the window means
    else:
        bytes_ = n * (2 * q * s + a)
    out = {"primal": q, "window": 8 + (1 if case["cs"] > 0 else 0), "adjoint": 1, "autograd": 1, "query": q + 4}[kind]
    return {"bytes": float(bytes_ + 8 * out * n), "flops": float(flops)}


# --------------------------------------------------------------------------
# the same in plain float64
# --------------------------------------------------------------------------

_C2 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 0), (-1, 1, 0)]
_C3 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1), (0, 1, 1), (0, 1, -1)]


class _Exact:
    """Populations as [q, nz, ny, nx] float64; the collision is cell-local, on [q, m]."""

    def __init__(self, s: _Setup, d):
        self.s, self.d = s, d
        half = _C2 if s.dim == 2 else _C3
        self.c = half + [tuple(-v for v in x) for x in half[1:]]
        self.q = len(self.c)
        h = (self.q - 1) // 2
        self.opp = [0] + list(range(h + 1, self.q)) + list(range(1, h + 1))
        w0, w1, w2 = (4 / 9, 1 / 9, 1 / 36) if s.dim == 2 else (1 / 3, 1 / 18, 1 / 36)
        self.w = [(w0, w1, w2)[sum(abs(v) for v in x)] for x in self.c]
        self.kS = 18.0 * math.sqrt(2.0) * s.cs * s.cs
        self.inlet = self.equilibrium(torch.ones(s.ny, device=DEV, dtype=torch.float64),
                                      [s.inflow(), 0.0 * s.inflow(), 0.0 * s.inflow()])[:, None, :]

    def equilibrium(self, rho, v, third=False):
        vv = v[0] * v[0] + v[1] * v[1] + v[2] * v[2]
        f = []
        for c, w in zip(self.c, self.w):
            cu = c[0] * v[0] + c[1] * v[1] + c[2] * v[2]
            e = 1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * vv
            if third:
                for a, b in self.third():
                    e = e + 13.5 * c[b] * (c[a] * c[a] - 1.0 / 3.0) * v[a] * v[a] * v[b]
            f.append(w * rho * e)
        return torch.stack(f)

    def third(self):
        return [(a, b) for a in range(self.s.dim) for b in range(self.s.dim) if a != b]

    def moments(self, f):
        rho = f.sum(0)
        j = [sum((c[a] * f[k] for k, c in enumerate(self.c) if c[a]), torch.zeros_like(rho)) for a in range(3)]
        return rho, j

    def flux(self, f, rho, j):
        """Non-equilibrium momentum flux with respect to the equilibrium at (rho, j / rho)."""
        P = {}
        for a in range(self.s.dim):
            for b in range(a, self.s.dim):
                m = sum(c[a] * c[b] * f[k] for k, c in enumerate(self.c) if c[a] * c[b])
                P[a, b] = m - (rho / 3.0 if a == b else 0.0) - j[a] * j[b] / rho
        return P

    @staticmethod
    def square(P):
        return sum((1.0 if a == b else 2.0) * v * v for (a, b), v in P.items())

    def tau_eff(self, f, rho, j, tau0):
        norm = torch.sqrt(self.square(self.flux(f, rho, j)) + 1e-60)
        return 0.5 * (tau0 + torch.sqrt(tau0 * tau0 + self.kS * norm))

    def collide(self, f, d, tau0, tau=None):
        """Cell-local collision; `tau` (a tensor or a number) where the relaxation time is frozen."""
        rho, j = self.moments(f)
        if tau is None:
            tau = self.tau_eff(f, rho, j, tau0) if self.s.cs > 0 else tau0
        om = 1.0 / tau
        v = [d * x / rho for x in j]
        if not self.s.hrr:
            return f + om * (self.equilibrium(rho, v) - f)
        a2 = {}
        for a in range(self.s.dim):
            for b in range(a, self.s.dim):
                m = sum(c[a] * c[b] * f[k] for k, c in enumerate(self.c) if c[a] * c[b])
                a2[a, b] = a2[b, a] = m - (rho / 3.0 if a == b else 0.0) - rho * v[a] * v[b]
        one = []
        for c, w in zip(self.c, self.w):
            g = sum(3.0 * c[a] * (1.0 - d) * j[a] for a in range(self.s.dim))
            for a in range(self.s.dim):
                for b in range(self.s.dim):
                    g = g + 4.5 * (c[a] * c[b] - (1.0 / 3.0 if a == b else 0.0)) * a2[a, b]
            for a, b in self.third():
                g = g + 13.5 * c[b] * (c[a] * c[a] - 1.0 / 3.0) * (2.0 * v[a] * a2[a, b] + v[b] * a2[a, a])
            one.append(w * g)
        return self.equilibrium(rho, v, third=True) + (1.0 - om) * torch.stack(one)

    def virtual(self, f_last):
        """Density-1 equilibrium at the velocity of the last column: what the outlet's virtual
        column sends back."""
        rho, j = self.moments(f_last)
        return self.equilibrium(torch.ones_like(rho), [x / rho for x in j])

    def stream(self, c, v):
        """c [q, nz, ny, nx] post-collision, v [q, nz, ny] the virtual column."""
        s, out = self.s, []
        for k, (cx, cy, cz) in enumerate(self.c):
            g = torch.roll(c[k], (cz, cy, cx), (0, 1, 2))
            if cx == -1:
                g = torch.cat([g[..., :-1], torch.roll(v[k], (cz, cy), (0, 1))[..., None]], -1)
            if s.walls and cy:  # halfway bounce-back
                o = c[self.opp[k]]
                g = torch.cat([o[:, :1], g[:, 1:]], 1) if cy > 0 else torch.cat([g[:, :-1], o[:, -1:]], 1)
            out.append(torch.cat([self.inlet[k].expand(s.nz, s.ny)[..., None], g[..., 1:]], -1))
        return torch.stack(out)

    def local(self, fn, f, *fields):
        """fn over the cells in pieces (memory)."""
        f = f.reshape(self.q, -1)
        m = 1 << 21
        parts = [fn(f[:, i:i + m], *[x.reshape(-1)[i:i + m] if torch.is_tensor(x) else x for x in fields])
                 for i in range(0, f.shape[1], m)]
        return torch.cat(parts, -1)

    def step(self, f):
        s = self.s
        c = self.local(lambda g, d: self.collide(g, d, s.tau), f, self.d).view_as(f)
        c[..., 0] = self.inlet
        return self.stream(c, self.virtual(f[..., -1]))

    def start(self, u):
        s = self.s
        v = [self.d * x for x in u.view(3, s.nz, s.ny, s.nx)]
        f = self.equilibrium(torch.ones_like(self.d), v)
        f[..., 0] = self.inlet
        return f

    # objective over the region: value per cell, from [q, ...] and d
    def density(self, f, d):
        s = self.s
        rho, j = self.moments(f)
        if s.kind == H.OBJ_FFA:
            return j[0] * s.u_max - j[0] * j[0] / rho + 1.0 / 3.0 - rho / 3.0
        nu = (s.tau - 0.5) / 3.0
        uu = sum(x * x for x in j) / (rho * rho)
        return 9.0 * nu / (2.0 * s.tau * s.tau) * self.square(self.flux(f, rho, j)) + (1.0 - d) / s.tau * uu

    def region(self, t):
        lo, hi = self.s.lo, self.s.hi
        return t[..., lo[2]:hi[2] + 1, lo[1]:hi[1] + 1, lo[0]:hi[0] + 1]

    def J(self, f):
        return self.density(self.region(f), self.region(self.d)).sum()

    def partials(self, f):
        """J, dJ/df and dJ/dd over the region."""
        with torch.enable_grad():
            g = self.region(f).clone().requires_grad_(True)
            d = self.region(self.d).clone().requires_grad_(True)
            J = self.density(g, d).sum()
            a, b = torch.autograd.grad(J, (g, d), allow_unused=True)
        return J.detach(), a, torch.zeros_like(d) if b is None else b

    def window(self, f, steps):
        """Means over `steps` samples (the state each step reads) and the state after them."""
        s = self.s
        m = {"f": torch.zeros_like(f), "J": 0.0, "gf": 0.0, "gd": 0.0, "tau": torch.zeros_like(self.d)}
        for _ in range(steps):
            J, a, b = self.partials(f)
            m["f"] += f / steps
            for k, v in (("J", J), ("gf", a), ("gd", b)):
                m[k] = m[k] + v / steps
            if s.cs > 0:
                m["tau"] += self.local(lambda g: self.tau_eff(g, *self.moments(g), s.tau), f).view_as(self.d) / steps
            f = self.step(f)
        return f, m

    def steady(self, f):
        J, a, b = self.partials(f)
        tau = self.local(lambda g: self.tau_eff(g, *self.moments(g), self.s.tau), f).view_as(self.d) if self.s.cs > 0 else None
        return {"f": f, "J": J, "gf": a, "gd": b, "tau": tau}

    def gradient(self, m, iters):
        """lambda_1 = -g, lambda_k+1 = (dF/df)^T lambda_k - g; dJ/dd - lambda . dF/dd, with F the
        step at the frozen state m."""
        s, f = self.s, m["f"].clone()
        f[..., 0] = self.inlet
        ta = s.tau_adj
        tau = None if (s.cs > 0 and s.diff) else (ta + (m["tau"] - s.tau) if s.cs > 0 else ta)

        def transpose(phi, wrt_d):
            def piece(g, p, d, t):
                with torch.enable_grad():
                    x = (d if wrt_d else g).clone().requires_grad_(True)
                    c = self.collide(g, x, ta, t) if wrt_d else self.collide(x, d, ta, t)
                    return torch.autograd.grad(c, x, p)[0].reshape(1 if wrt_d else self.q, -1)
            g, p, out, step = f.reshape(self.q, -1), phi.reshape(self.q, -1), [], 1 << 20
            for i in range(0, g.shape[1], step):
                t = tau.reshape(-1)[i:i + step] if torch.is_tensor(tau) else tau
                out.append(piece(g[:, i:i + step], p[:, i:i + step], self.d.reshape(-1)[i:i + step], t))
            out = torch.cat(out, -1).view((1 if wrt_d else self.q, s.nz, s.ny, s.nx))
            out[..., 0] = 0.0  # the inlet is pinned
            return out

        lam = torch.zeros_like(f)
        phi = torch.zeros_like(f)
        pv = torch.zeros(self.q, s.nz, s.ny, device=DEV, dtype=torch.float64)
        zero, zero_v = torch.zeros_like(f), torch.zeros_like(pv)
        for _ in range(iters):
            lam = transpose(phi, False)
            with torch.enable_grad():
                last = f[..., -1].clone().requires_grad_(True)
                lam[..., -1] += torch.autograd.grad(self.virtual(last), last, pv)[0]
            self.region(lam).sub_(m["gf"])
            with torch.enable_grad():  # the streaming is linear: its transpose from its own derivative
                a, b = zero.requires_grad_(True), zero_v.requires_grad_(True)
                phi, pv = torch.autograd.grad(self.stream(a, b), (a, b), lam)
            phi[..., 0] = 0.0
        out = -transpose(phi, True)[0]
        self.region(out).add_(m["gd"])
        return out


def _flat(t):
    return t.reshape(-1)


def _vector(j, rho):
    return torch.stack([x / rho for x in j]).reshape(-1)


def _mean_fields(E, m):
    rho, j = E.moments(m["f"])
    rho[..., 0] = 1.0  # the pinned inlet takes no part in the window
    for x in j:
        x[..., 0] = 0.0
    return _flat(rho), _vector(j, rho)


def exact(case, seed):
    kind = case["kind"]
    if kind == "group":
        outs = []
        for k in range(case["members"]):
            c, mode = _member(case, k)
            s = _Setup(c, seed * 64 + k)
            noise, u = s.fields()
            E = _Exact(s, s.porosity(noise))
            f = E.start(u)
            if mode == H.GROUP_PRIMAL:
                for _ in range(case["steps"]):
                    f = E.step(f)
                outs.append({"populations": _flat(f)})
            elif mode == H.GROUP_PRIMAL_WINDOW:
                f, m = E.window(f, case["steps"])
                rho, u = _mean_fields(E, m)
                outs.append({"populations": _flat(f), "mean_rho": rho, "mean_u": u})
            else:
                outs.append({"gradient": _flat(E.gradient(E.steady(f), case["steps"]))})
        return outs
    if case["diff"] and case["dim"] == 3 and case["nx"] * case["ny"] * case["nz"] > 8_000_000:
        return None
    s = _Setup(case, seed)
    noise, u = s.fields()
    E = _Exact(s, s.porosity(noise))
    if kind == "autograd":
        f = E.start(u)
        for _ in range(case["steps"]):
            f = E.step(f)
        m = E.steady(f)
        return {"J": m["J"], "gradient": _flat(E.gradient(m, case["adjoint"]))}
    f = E.start(u)
    del noise, u
    if kind == "primal":
        probe, at = [], (min(s.nx - 2, int(s.xc + 2 * s.D)), int(s.yc), s.nz // 2)
        for _ in range(case["steps"]):
            if case["probe"]:
                rho, j = E.moments(f[:, at[2], at[1], at[0]])
                probe.append(j[1] / rho)
            f = E.step(f)
        r = {"populations": _flat(f), "J": E.J(f)}
        if case["probe"]:
            r["probe"] = torch.stack(probe)
        return r
    if kind != "adjoint":
        for _ in range(case["steps"]):
            f = E.step(f)
    f, m = E.window(f, case["window"])
    mean_rho, mean_u = _mean_fields(E, m)
    if kind == "window":
        rho, j = E.moments(f)
        r = {"rho": _flat(rho), "u": _vector(j, rho), "mean_rho": mean_rho, "mean_u": mean_u, "J": m["J"]}
        if s.cs > 0:
            m["tau"][..., 0] = 0.0
            r["mean_tau"] = _flat(m["tau"])
        return r
    r = {"gradient": None, "J": m["J"]}
    if kind == "query":
        r.update(populations=_flat(f), mean_u=mean_u)
        del f
    r["gradient"] = _flat(E.gradient(m, case["adjoint"]))
    return r
