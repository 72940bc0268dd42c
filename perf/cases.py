"""The workloads whose time is measured: what a user of this framework has it
do, through its public entry points, with the sizes of the benchmark, the
tests and the closure experiment.

listed() names them; draw() gives further ones of the same ranges; prepare()
makes the inputs and the handle that a program keeps; run() is one pass; work()
is what a pass cannot do without; exact() is the same pass in 64 bits, written
with plain torch from the scheme's equations.

A pass advances the state it was given, so the next pass continues from there.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2012_03525_amd import acm, closure, inputs

DEV = "cuda:0"
PER, WALL, SYM = acm.PERIODIC, acm.WALL, acm.SYMMETRY
NAMES = ("drho", "u", "v", "w", "phi")

# operations per node and step (adds, multiplies and fused multiply-adds as
# two), counted from the scheme: continuity, fluxes, Laplacians, SATs, update
FLOPS = {"flow2d": 110, "flow3d": 230, "drop2d": 260, "drop3d": 550, "pipe": 140, "drop_axis": 320}
# multiply-adds of the five 3x3 layers 3-32-32-32-32-3, per node
NET_FLOPS = 2 * 9 * (3 * 32 + 3 * 32 * 32 + 32 * 3)


def listed():
    return [
        # the paper's first test at its smallest size: 64 x 64 doubles, 100
        # steps with the default options; launches and latency are all there is
        {"name": "tgv2d_64_f64", "kind": "flow2d", "nx": 64, "ny": 64, "prec": "f64", "faces": "periodic",
         "nu": 0.01, "u0": 0.01, "steps": 100, "fine": False},
        # the closure's fine reference: forced periodic flow on 1024 x 1024,
        # configured as the closure experiment does, one gate interval / 4
        {"name": "forced2d_1024", "kind": "flow2d", "nx": 1024, "ny": 1024, "prec": "f32", "faces": "periodic",
         "nu": 0.02, "u0": 0.03, "steps": 100, "fine": True},
        # a lid-driven cavity with sides that divide by nothing
        {"name": "cavity2d_401x257", "kind": "flow2d", "nx": 401, "ny": 257, "prec": "f32", "faces": "cavity",
         "nu": 0.02, "u0": 0.05, "steps": 150, "fine": False},
        # the benchmark's headline: 3D Taylor-Green 256^3, single precision
        {"name": "tgv3d_256", "kind": "flow3d", "nx": 256, "ny": 256, "nz": 256, "prec": "f32", "faces": "periodic",
         "nu": 0.05 * (256 / (2 * math.pi)) / 1600.0, "u0": 0.05, "steps": 20},
        # a body-forced duct between walls, three different odd-sized axes
        {"name": "duct3d_200x99x70", "kind": "flow3d", "nx": 200, "ny": 99, "nz": 70, "prec": "f32", "faces": "duct",
         "nu": 0.02, "u0": 0.05, "steps": 40},
        # two phases in 2D: the drop in shear between moving walls
        {"name": "drop_shear_1024", "kind": "drop2d", "nx": 1024, "ny": 1024, "prec": "f32", "steps": 64},
        # two phases in 3D with a wetting wall: the drop spreading on a wall
        {"name": "drop_spreading_96", "kind": "drop3d", "n": 96, "prec": "f32", "theta": 60.0, "steps": 64},
        # the axisymmetric step on the largest 2D grid the benchmark has
        {"name": "pipe_4096x2048", "kind": "pipe", "nx": 4096, "ny": 2048, "prec": "f32", "steps": 64},
        # the axisymmetric two-phase step
        {"name": "drop_axis_2048x1024", "kind": "drop_axis", "nx": 2048, "ny": 1024, "prec": "f32", "steps": 64},
        # the serving-style sweep: 512 uneven cases, one 500-step chunk
        {"name": "batch_512", "kind": "batch", "cases": 512, "smallest": 32, "largest": 256, "mix": 4, "chunk": 500},
        # the learned closure between two gates: 100 corrected coarse steps,
        # then the diagnostics that the gate reads
        {"name": "closure_256", "kind": "closure", "n": 256, "steps": 100},
        # one step of training the closure through two solver steps, with the
        # divergence penalty: network forward and backward, step adjoint, Adam
        {"name": "train_256_k2", "kind": "train", "n": 256, "k": 2, "beta": 3.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["flow2d", "flow2d", "flow3d", "flow3d", "drop2d", "drop3d", "pipe", "drop_axis", "batch",
                       "closure", "train"])
    prec = "f64" if rng.random() < 0.25 else "f32"
    steps = _log_int(rng, 16, 100)
    if kind == "flow2d":
        return {"kind": kind, "nx": _log_int(rng, 24, 2048), "ny": _log_int(rng, 24, 2048), "prec": prec,
                "faces": rng.choice(["periodic", "duct", "cavity"]), "nu": round(rng.uniform(0.01, 0.05), 4),
                "u0": 0.03, "steps": steps, "fine": False}
    if kind == "flow3d":
        return {"kind": kind, "nx": rng.choice([64, 128, 256, _log_int(rng, 24, 200), _log_int(rng, 24, 200)]),
                "ny": _log_int(rng, 24, 200), "nz": _log_int(rng, 24, 160), "prec": prec,
                "faces": rng.choice(["periodic", "duct", "cavity"]), "nu": round(rng.uniform(0.01, 0.05), 4),
                "u0": 0.03, "steps": min(steps, 32)}
    if kind == "drop2d":
        return {"kind": kind, "nx": _log_int(rng, 64, 1024), "ny": _log_int(rng, 64, 1024), "prec": prec,
                "steps": min(steps, 64)}
    if kind == "drop3d":
        return {"kind": kind, "n": _log_int(rng, 32, 96), "prec": prec, "theta": float(rng.choice([45, 60, 90, 120])),
                "steps": min(steps, 40)}
    if kind == "pipe":
        return {"kind": kind, "nx": _log_int(rng, 64, 4096), "ny": _log_int(rng, 32, 2048), "prec": prec,
                "steps": min(steps, 64)}
    if kind == "drop_axis":
        return {"kind": kind, "nx": _log_int(rng, 96, 2048), "ny": _log_int(rng, 64, 1024), "prec": prec,
                "steps": min(steps, 64)}
    if kind == "batch":
        return {"kind": kind, "cases": _log_int(rng, 16, 256), "smallest": 32, "largest": rng.choice([96, 160, 256]),
                "mix": rng.randrange(1000), "chunk": 2 * _log_int(rng, 25, 150)}
    if kind == "closure":
        return {"kind": kind, "n": 64 * rng.randint(1, 6), "steps": _log_int(rng, 20, 200)}
    return {"kind": kind, "n": 64 * rng.randint(1, 5), "k": rng.randint(1, 3), "beta": rng.choice([0.0, 3.0])}


# ---------------------------------------------------------------------------
# problem set-up
# ---------------------------------------------------------------------------
def _faces(dim, name):
    """Boundary types and wall velocities of the six faces."""
    wu = [[0.0] * 3 for _ in range(6)]
    if name == "periodic":
        return [PER] * 6, wu
    if name == "duct":
        return [PER, PER, WALL, WALL] + ([WALL, WALL] if dim == 3 else [PER, PER]), wu
    wu[2 * dim - 1][0] = 0.05
    return [WALL] * 4 + ([WALL, WALL] if dim == 3 else [PER, PER]), wu


def _problem(case):
    """make_config keywords of a solver case (dim, sizes, faces, coefficients)."""
    kind = case["kind"]
    if kind in ("flow2d", "flow3d"):
        dim = 2 if kind == "flow2d" else 3
        bc, wu = _faces(dim, case["faces"])
        g = (1e-6, 0.0, 0.0) if case["faces"] == "duct" else (0.0, 0.0, 0.0)
        p = dict(dim=dim, nx=case["nx"], ny=case["ny"], nz=case.get("nz", 1), nu=case["nu"], bc=bc, wall_u=wu, g=g)
    elif kind == "drop2d":
        _, wu = _faces(2, "periodic")
        wu[2][0], wu[3][0] = -0.02, 0.02
        p = dict(dim=2, nx=case["nx"], ny=case["ny"], nz=1, nu=1.0 / 6.0, bc=[PER, PER, WALL, WALL, PER, PER],
                 wall_u=wu, two_phase=True, sigma=0.01, width=4.0, mobility=0.02)
    elif kind == "drop3d":
        n = case["n"]
        size, c, re, cn, pe = n / 3.0, 10.0, 100.0, 0.1, 8000.0
        nu = size / (c * re)
        wet = [0.0] * 6
        wet[4] = math.cos(math.radians(case["theta"]))
        p = dict(dim=3, nx=n, ny=n, nz=n, nu=nu, bc=[SYM] * 4 + [WALL] * 2, two_phase=True,
                 sigma=size / (c * c * re), width=max(cn * size, 2.0), mobility=size * size / (pe * nu), wet_cos=wet)
    elif kind == "pipe":
        p = dict(dim=2, nx=case["nx"], ny=case["ny"], nz=1, nu=0.05, bc=[PER, PER, SYM, WALL, PER, PER],
                 g=(4 * 0.05 * 0.05 / case["ny"] ** 2, 0.0, 0.0), axisym=True)
    elif kind == "drop_axis":
        p = dict(dim=2, nx=case["nx"], ny=case["ny"], nz=1, nu=0.1, bc=[PER, PER, SYM, SYM, PER, PER], axisym=True,
                 two_phase=True, sigma=0.01, width=4.0, mobility=0.1)
    p.setdefault("wall_u", [[0.0] * 3 for _ in range(6)])
    p.setdefault("g", (0.0, 0.0, 0.0))
    p.setdefault("wet_cos", [0.0] * 6)
    return p


def _axes(p):
    """Cell-centre coordinates in [0, 1), shaped to broadcast over the grid."""
    sizes = (p["nx"], p["ny"], p["nz"])[:p["dim"]]
    out = []
    for a, n in enumerate(sizes):
        shape = [1] * p["dim"]
        shape[-1 - a] = n
        out.append(((torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n).reshape(shape))
    return out


def _phases(seed, n=16):
    return (2 * math.pi * np.random.Generator(np.random.PCG64(seed)).random(n)).tolist()


def _vortices(p, seed, amp):
    """Taylor-Green-like vortices with seeded phases, zero at walls, and the
    density of their pressure."""
    ph = _phases(seed)
    x = [2 * math.pi * c for c in _axes(p)]
    X, Y = x[0] + ph[0], x[1] + ph[1]
    Z = x[2] + ph[2] if p["dim"] == 3 else torch.zeros_like(X)
    u = amp * torch.sin(X) * torch.cos(Y) * torch.cos(Z)
    v = -amp * torch.cos(X) * torch.sin(Y) * torch.cos(Z)
    w = 0.1 * amp * torch.cos(X + ph[3]) * torch.cos(Y + ph[4]) * torch.ones_like(Z)
    for a, c in enumerate(x):
        if p["bc"][2 * a] != PER:
            u, v, w = (f * torch.sin(0.5 * c) ** 2 for f in (u, v, w))
    r = 3.0 * amp * amp / 16.0 * (torch.cos(2 * X) + torch.cos(2 * Y)) * (torch.cos(2 * Z) + 2.0)
    return {"drho": r, "u": u, "v": v, "w": w}


def _initial(case, p, seed):
    """The initial fields in the case's precision."""
    kind, ph = case["kind"], _phases(seed)
    full = tuple((p["nx"], p["ny"], p["nz"])[:p["dim"]][::-1])
    if kind in ("flow2d", "flow3d"):
        s = _vortices(p, seed, case["u0"])
        if case["kind"] == "flow2d" and case["fine"]:
            f = inputs.random_spectrum_field(case["nx"], seed, case["u0"])
            s = {k: torch.from_numpy(a).to(DEV) for k, a in f.items()}
    elif kind == "pipe":
        x, y = _axes(p)
        tp = 2 * math.pi
        s = {"u": 0.04 * (1 - y * y) * (1 + 0.3 * torch.sin(tp * x + ph[0])),
             "v": 0.008 * y * (1 - y) * torch.sin(tp * x + ph[1]),
             "drho": 1e-3 * torch.cos(tp * x + ph[2]) * torch.cos(math.pi * y)}
    else:
        s = _vortices(p, seed, 0.002)
        x = [c * n for c, n in zip(_axes(p), (p["nx"], p["ny"], p["nz"]))]
        if kind == "drop2d":
            s["u"] = s["u"] + 0.02 * (2 * _axes(p)[1] - 1)
            radius, centre = min(p["nx"], p["ny"]) / 8.0, (p["nx"] / 2 + ph[5] / 3, p["ny"] / 2 + ph[6] / 3)
        elif kind == "drop3d":
            radius, centre = p["nx"] / 3.0 + ph[5] / 6, (0.0, 0.0, 0.0)
        else:
            s["v"] = s["v"] * torch.sin(math.pi * _axes(p)[1])
            radius, centre = p["ny"] / 4.0, (p["nx"] / 2 + ph[5] / 3, 0.0)
        d = sum((c - c0) ** 2 for c, c0 in zip(x, centre)).sqrt()
        s["phi"] = torch.tanh(2.0 * (radius - d) / p["width"])
    dt = torch.float64 if case["prec"] == "f64" else torch.float32
    names = [k for k in NAMES if k in s and (k != "w" or p["dim"] == 3)]
    return {k: s[k].expand(full).to(dt).contiguous() for k in names}


def _force(case):
    """Kolmogorov forcing of the fine reference, else none."""
    if case["kind"] == "flow2d" and case["fine"]:
        return closure.FlowSpec(n_fine=case["nx"], nu_fine=case["nu"]).fine_force()
    return None


def _batch_geometry(case):
    sizes = tuple(range(case["smallest"], case["largest"] + 1, 16))
    geo = inputs.batch_cases(case["cases"], seed=case["mix"], sizes=sizes, chunk=case["chunk"], with_state=False)
    for c in geo:
        c.nu = max(c.nu, 0.04)  # no case diverges, so every pass has the whole sweep to do
    return geo


def _batch_state(c, seed):
    walls = c.kind == "cavity"
    pert = inputs.low_mode_perturbation(c.n, seed % 100003 * 1009 + c.index, 1e-3, walls=walls)
    s = {k: np.zeros((c.n, c.n)) for k in ("drho", "u", "v")} if walls else inputs.tgv2d(c.n, c.u_ref)
    return {"drho": s["drho"], "u": s["u"] + pert["u"], "v": s["v"] + pert["v"]}


IN_SCALE, OUT_SCALE = (3000.0, 50.0, 50.0), (0.0, 1e-6, 1e-6)


def _coarse(case, seed):
    """A coarse state with the closure's initial spectrum, single precision."""
    n = case["n"]
    f = inputs.random_spectrum_field(n, seed, 0.03, kmax=min(16, n // 8))
    return {k: torch.from_numpy(a).to(DEV, torch.float32) for k, a in f.items()}


def _spec(case):
    return closure.FlowSpec(n_fine=4 * case["n"])


def _targets(case, q0, seed):
    """States the corrected steps are trained towards: the plain coarse
    steps plus a smooth residual of the size of the output scale."""
    spec, n = _spec(case), case["n"]
    P = _Step(dict(dim=2, nx=n, ny=n, nz=1, nu=spec.nu_fine / spec.ratio, bc=[PER] * 6, g=(0, 0, 0)),
              torch.from_numpy(spec.coarse_force()).to(DEV))
    q, out = {k: t.double() for k, t in q0.items()}, []
    for j in range(case["k"]):
        q = P.step(q)
        e = inputs.random_spectrum_field(n, seed + 77 + j, OUT_SCALE[1], kmax=min(16, n // 8))
        out.append({k: (q[k] + torch.from_numpy(e[k]).to(DEV)).float() for k in q})
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        geo = _batch_geometry(case)
        cfgs = []
        for c in geo:
            bc, wu = _faces(2, "cavity" if c.kind == "cavity" else "periodic")
            cfgs.append(acm.make_config(2, c.n, c.n, nu=c.nu, precision="f32", bc=bc, wall_u=wu))
        # a sweep long enough that no case retires while it is measured
        b = acm.Batch(cfgs, [_batch_state(c, seed) for c in geo], [10 ** 9] * len(geo), chunk=case["chunk"])
        # where the newest states (set a) lie in the arena, to collect them
        pos = [torch.arange(int(o), int(o) + 3 * c.n * c.n, device=DEV) for o, c in zip(b.offsets, geo)]
        return {"kind": kind, "batch": b, "pos": torch.cat(pos)}
    if kind == "closure":
        net = closure.Network(case["n"], case["n"], seed=seed, in_scale=IN_SCALE, out_scale=OUT_SCALE)
        return {"kind": kind, "run": closure.ClosureRun(_spec(case), net, _coarse(case, seed)), "steps": case["steps"]}
    if kind == "train":
        net = closure.Network(case["n"], case["n"], seed=seed, in_scale=IN_SCALE, out_scale=OUT_SCALE)
        q0 = _coarse(case, seed)
        return {"kind": kind, "net": net, "un": closure.Unroll(_spec(case), net, case["k"], case["beta"]), "q0": q0,
                "targets": _targets(case, q0, seed)}
    p = _problem(case)
    a = _initial(case, p, seed)
    if kind == "flow2d" and case["fine"]:
        cfg = closure.FlowSpec(n_fine=case["nx"], nu_fine=case["nu"]).fine_config()
    else:
        dims = [p.pop(k) for k in ("dim", "nx", "ny", "nz")]
        cfg = acm.make_config(*dims, precision=case["prec"], **p)
    sets = [a, {k: torch.empty_like(t) for k, t in a.items()}]
    return {"kind": kind, "solver": acm.Solver(cfg, None, tensors=sets, force_x=_force(case)), "steps": case["steps"]}


def run(state):
    kind = state["kind"]
    if kind == "batch":
        b = state["batch"]
        b.run(1)
        return torch.index_select(b.arena, 0, state["pos"])
    if kind == "closure":
        r = state["run"]
        r.run(state["steps"])
        d = r.diagnostics()
        return {"state": dict(r.state()), "ke": d["ke"], "enstrophy": d["enstrophy"], "div_rms": d["div_rms"]}
    if kind == "train":
        net = state["net"]
        loss = state["un"].train_step(state["q0"], state["targets"], 1e-4)
        return {"loss": loss, "gw": list(net.gw), "gb": list(net.gb)}
    s = state["solver"]
    s.run(state["steps"])
    return dict(s.tensors())


def work(case):
    """Each input read once, each output written once, and the arithmetic."""
    kind = case["kind"]
    if kind == "batch":
        nodes = sum(c.n * c.n for c in _batch_geometry(case))
        return {"bytes": 24 * nodes, "flops": case["chunk"] * nodes * FLOPS["flow2d"]}
    if kind == "closure":
        nodes = case["n"] ** 2
        return {"bytes": 24 * nodes, "flops": case["steps"] * nodes * (NET_FLOPS + FLOPS["flow2d"])}
    if kind == "train":
        nodes = case["n"] ** 2
        # per step: network forward, data and weight gradients; step and adjoint
        return {"bytes": 12 * nodes * (1 + case["k"]), "flops": case["k"] * nodes * (3 * NET_FLOPS + 300)}
    p = _problem(case)
    nodes = p["nx"] * p["ny"] * p["nz"]
    fields = (3 if p["dim"] == 2 else 4) + (1 if p.get("two_phase") else 0)
    size = 8 if case["prec"] == "f64" else 4
    return {"bytes": 2 * fields * size * nodes, "flops": case["steps"] * nodes * FLOPS[kind]}


# ---------------------------------------------------------------------------
# the same passes in 64 bits
# ---------------------------------------------------------------------------
class _Step:
    """One step in double precision: Eqs. (2.10)-(2.13), two-phase with Heun's
    method for Eq. (2.14), cylindrical operators when axisymmetric; dx = dt =
    rho0 = 1, cs^2 = 1/3.  Fields may have leading batch axes; nu broadcasts."""

    def __init__(self, p, force=None):
        self.p, self.dim, self.bc = p, p["dim"], p["bc"]
        self.wall_u = p.get("wall_u") or [[0.0] * 3 for _ in range(6)]
        self.force = force.reshape(-1, 1) if force is not None else 0.0
        self.nu, self.axi, self.two = p["nu"], p.get("axisym", False), p.get("two_phase", False)
        if self.axi:
            self.row = torch.arange(p["ny"], device=DEV, dtype=torch.float64).reshape(-1, 1)
            self.ir = 1.0 / (self.row + 0.5)
        if self.two:
            self.a4 = 3.0 * p["sigma"] / p["width"]
            self.kappa = 3.0 * p["sigma"] * p["width"] / 8.0
            self.wet = [2.0 / p["width"] * c if b == WALL else 0.0 for c, b in zip(p["wet_cos"], self.bc)]

    def ghost(self, m, face, comp, wet):
        bc = self.bc[face]
        if comp is not None:
            if bc == WALL:
                return 2.0 * self.wall_u[face][comp] - m
            return -m if comp == face // 2 else m
        if wet and self.wet[face]:
            b, mc = self.wet[face], m.clamp(-1.0, 1.0)
            q = 2.0 * mc + b
            return m + 2.0 * (q / (1.0 + (1.0 + b * q).sqrt()) - mc)
        return m

    def ext(self, f, comp=None, wet=False):
        """One ghost layer around f, faces in x, y, z order."""
        for a in range(self.dim):
            ax = f.dim() - 1 - a
            first, last = f.narrow(ax, 0, 1), f.narrow(ax, f.shape[ax] - 1, 1)
            if self.bc[2 * a] == PER:
                lo, hi = last, first
            else:
                lo, hi = self.ghost(first, 2 * a, comp, wet), self.ghost(last, 2 * a + 1, comp, wet)
            f = torch.cat([lo, f, hi], ax)
        return f

    def at(self, F, *off):
        """Inner part of an extended field, shifted by (axis, offset) pairs."""
        d = [0] * self.dim
        for a, s in off:
            d[a] += s
        for a in range(self.dim):
            ax = F.dim() - 1 - a
            F = F.narrow(ax, 1 + d[a], F.shape[ax] - 2)
        return F

    def diff(self, F, a):
        return self.at(F, (a, 1)) - self.at(F, (a, -1))

    def lap(self, F):
        if self.axi:
            c, n, s = self.at(F), self.at(F, (1, 1)), self.at(F, (1, -1))
            return (self.at(F, (0, 1)) + self.at(F, (0, -1)) - 2 * c) + (self.row * (n + s - 2 * c) + (n - c)) * self.ir
        return sum(self.at(F, (a, 1)) + self.at(F, (a, -1)) for a in range(self.dim)) - 2 * self.dim * self.at(F)

    def ddy(self, F):
        """y part of a divergence, times 2 dx (cylindrical when axisymmetric)."""
        if self.axi:
            return (self.row * self.diff(F, 1) + self.at(F) + self.at(F, (1, 1))) * self.ir
        return self.diff(F, 1)

    def grad_iso(self, F, a):
        g = (4.0 if self.dim == 2 else 2.0) * self.diff(F, a)
        for b in range(self.dim):
            if b != a:
                g = g + sum(self.at(F, (a, 1), (b, s)) - self.at(F, (a, -1), (b, s)) for s in (1, -1))
        return g / 12.0

    def lap_iso(self, F):
        w, c0 = (4.0, 20.0) if self.dim == 2 else (2.0, 24.0)
        t = w * sum(self.at(F, (a, s)) for a in range(self.dim) for s in (1, -1)) - c0 * self.at(F)
        for a in range(self.dim):
            for b in range(a):
                t = t + sum(self.at(F, (a, s), (b, r)) for s in (1, -1) for r in (1, -1))
        t = t / 6.0
        return t + self.ir * self.grad_iso(F, 1) if self.axi else t

    def step(self, q):
        D, nu = self.dim, self.nu
        r, vel = q["drho"], [q[k] for k in ("u", "v", "w")[:D]]
        R = self.ext(r)
        V = [self.ext(f, comp=a) for a, f in enumerate(vel)]
        M = [(1.0 + R) * f for f in V]
        div = sum(self.ddy(M[a]) if a == 1 else self.diff(M[a], a) for a in range(D))
        rn = r - 0.5 * div + self.lap(R) / 6.0
        RN = self.ext(rn)
        out = {"drho": rn}
        if self.two:
            phi, mob = q["phi"], self.p["mobility"]

            def mu_of(f, F):
                return self.a4 * f * (f * f - 1.0) - self.kappa * self.lap_iso(F)

            def rate(F, MU):
                return mob * self.lap_iso(MU) - sum(vel[a] * self.grad_iso(F, a) for a in range(D))
            PH = self.ext(phi, wet=True)
            MU = self.ext(mu_of(phi, PH))
            ps = phi + rate(PH, MU)
            PS = self.ext(ps, wet=True)
            out["phi"] = 0.5 * (phi + ps + rate(PS, self.ext(mu_of(ps, PS))))
        for a in range(D):
            flux = 0.0
            for b in range(D):
                F = M[a] * V[b] + (R / 3.0 if a == b else 0.0)
                flux = flux + (self.ddy(F) if b == 1 else self.diff(F, b))
            lap = self.lap(M[a])
            if self.axi and a == 1:
                flux = flux - 2.0 / 3.0 * r * self.ir
                lap = lap - self.at(M[a]) * self.ir * self.ir
            dm = -0.5 * flux + nu * lap - 0.5 * (nu + 1.0 / 6.0) * (self.diff(RN, a) - self.diff(R, a))
            dm = dm + (1.0 + rn) * (self.p["g"][a] + (self.force if a == 0 else 0.0))
            if self.two:
                dm = dm - phi * self.grad_iso(MU, a)
            out[("u", "v", "w")[a]] = (self.at(M[a]) + dm) / (1.0 + rn)
        return out


def _net_params(seed):
    out = []
    for w, b in closure.he_init(seed):
        w = torch.from_numpy(np.asarray(w, dtype=np.float32)).to(DEV).to(torch.bfloat16).double()
        out.append((w, torch.zeros(b.shape, device=DEV, dtype=torch.float64)))
    return out


def _network(q, params):
    """The five circular 3x3 layers on the scaled fields (3 channels out)."""
    x = torch.stack([s * q[k] for s, k in zip(IN_SCALE, ("drho", "u", "v"))], -1)
    for l, (w, b) in enumerate(params):
        h, wd, c = x.shape
        y = b
        for t in range(9):
            y = y + torch.roll(x, (1 - t // 3, 1 - t % 3), (0, 1)).reshape(-1, c) @ w[t].t()
        x = y.reshape(h, wd, -1)
        x = x.clamp_min(0.0) if l < len(params) - 1 else x
    return x


def _correct(s, params):
    raw = _network(s, params)
    return {k: s[k] + OUT_SCALE[c] * raw[..., c] for c, k in enumerate(("drho", "u", "v"))}


def _coarse_step(case):
    spec = _spec(case)
    f = torch.from_numpy(spec.coarse_force()).to(DEV, torch.float32).double()
    return _Step(dict(dim=2, nx=case["n"], ny=case["n"], nz=1, nu=spec.nu_fine / spec.ratio, bc=[PER] * 6,
                      g=(0, 0, 0)), f)


def _cdiv(u, v):
    """Centred periodic divergence, grid units."""
    return 0.5 * ((torch.roll(u, -1, 1) - torch.roll(u, 1, 1)) + (torch.roll(v, -1, 0) - torch.roll(v, 1, 0)))


def _exact_batch(case, seed):
    geo = _batch_geometry(case)
    done = [None] * len(geo)
    for key in sorted({(c.n, c.kind) for c in geo}):
        mine = [c for c in geo if (c.n, c.kind) == key]
        bc, wu = _faces(2, "cavity" if key[1] == "cavity" else "periodic")
        states = [_batch_state(c, seed) for c in mine]
        q = {k: torch.from_numpy(np.stack([s[k] for s in states])).to(DEV, torch.float32).double()
             for k in ("drho", "u", "v")}
        nu = torch.tensor([c.nu for c in mine], device=DEV, dtype=torch.float64).reshape(-1, 1, 1)
        P = _Step(dict(dim=2, nx=key[0], ny=key[0], nz=1, nu=nu, bc=bc, wall_u=wu, g=(0, 0, 0)))
        for _ in range(case["chunk"]):
            q = P.step(q)
        for i, c in enumerate(mine):
            done[c.index] = torch.cat([q[k][i].reshape(-1) for k in ("drho", "u", "v")])
    return torch.cat(done)


def _exact_train(case, seed):
    params = [(w.requires_grad_(), b.requires_grad_()) for w, b in _net_params(seed)]
    P, q0, k = _coarse_step(case), _coarse(case, seed), case["k"]
    targets = _targets(case, q0, seed)
    q, loss = {n: t.double() for n, t in q0.items()}, 0.0
    for j in range(k):
        s = P.step(q)
        q = _correct(s, params)
        e = [(q[n] - targets[j][n].double()) / OUT_SCALE[c] for c, n in ((1, "u"), (2, "v"))]
        loss = loss + sum((x * x).mean() for x in e) / 2 / k
        if case["beta"]:
            d = _cdiv(q["u"] - s["u"], q["v"] - s["v"])
            loss = loss + case["beta"] / OUT_SCALE[1] ** 2 / k * (d * d).mean()
    loss.backward()
    gw, gb = [], []
    for l, (w, b) in enumerate(params):
        ci, co = closure.layer_shape(l)
        g = torch.zeros((9, co, ci), device=DEV, dtype=torch.float64)
        g[:, :w.shape[1], :w.shape[2]] = w.grad
        h = torch.zeros(co, device=DEV, dtype=torch.float64)
        h[:b.shape[0]] = b.grad
        gw.append(g)
        gb.append(h)
    return {"loss": loss.detach().reshape(1), "gw": gw, "gb": gb}


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed)
    with torch.no_grad():
        if kind == "batch":
            return _exact_batch(case, seed)
        if kind == "closure":
            P, params = _coarse_step(case), _net_params(seed)
            q = {k: t.double() for k, t in _coarse(case, seed).items()}
            for _ in range(case["steps"]):
                q = _correct(P.step(q), params)
            u, v = q["u"], q["v"]
            om = 0.5 * ((torch.roll(v, -1, 1) - torch.roll(v, 1, 1)) - (torch.roll(u, -1, 0) - torch.roll(u, 1, 0)))
            d = _cdiv(u, v)
            return {"state": q, "ke": float(0.5 * (u * u + v * v).sum()), "enstrophy": float(0.5 * (om * om).mean()),
                    "div_rms": float((d * d).mean().sqrt())}
        p = _problem(case)
        dt = torch.float64 if case["prec"] == "f64" else torch.float32
        f = _force(case)
        P = _Step(p, None if f is None else torch.from_numpy(f).to(DEV, dt).double())
        q = {k: t.double() for k, t in _initial(case, p, seed).items()}
        for _ in range(case["steps"]):
            q = P.step(q)
        return q
