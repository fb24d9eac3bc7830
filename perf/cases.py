"""Performance cases: what programs that use this solver have it do, through its public entry points.

A case is one pass of a program's main loop on a prepared problem: RK4 marching ("march"),
marching with the steady-state checks of a solve ("steady"), several problems advanced together
("batch"), implicit time steps ("implicit") and a served set of requests ("serve").  Problems are the
Couette and cavity flows of the benchmark and the tests, on meshes of 8 to 128 elements a side,
polynomial orders 1 to 4, the 16-velocity Gauss-Hermite set or Newton-Cotes sets of 6 x 6 to 24 x 24
velocities, Kn from 0.1 to 10.  Initial states are smooth fields of density and velocity with seeded
modes.

exact() repeats a pass in plain torch in 64 bits: nodal DG on tensor Gauss-Lobatto elements, upwind
fluxes, diffuse walls, BGK collision with the second-order equilibrium, classical RK4.
"""
import math
import random
import types

import numpy as np
import torch

import paper_2012_13487_amd as dg

CFL = 0.2
LID = 0.1          # lid and plate speed
NC_VMAX = 4.0      # Newton-Cotes sets span [-4, 4] in units of sqrt(RT)


# ---- the cases ----------------------------------------------------------------------------------

def march(name, flow, nx, ny, p, vel, precision, steps, graph=0, kn=1.0):
    return {"name": name, "kind": "march", "flow": flow, "nx": nx, "ny": ny, "p": p, "vel": vel,
            "precision": precision, "steps": steps, "graph": graph, "kn": kn}


def listed():
    return [
        # the smallest problem (9216 values): launches and latency, ordinary and replayed from a graph
        march("couette_8x8_p2_gh4", "couette", 8, 8, 2, "gh4", "fp64", 20),
        march("couette_8x8_p2_gh4_graph", "couette", 8, 8, 2, "gh4", "fp64", 50, graph=10),
        # a Couette flow of the mixed batch's largest mesh with the 16-velocity set: few velocities,
        # many elements
        march("couette_96x96_p2_gh4", "couette", 96, 96, 2, "gh4", "fp64", 10, kn=0.5),
        # the benchmark's headline problem
        march("cavity_64x64_p3_nc16", "cavity", 64, 64, 3, "nc16", "fp64", 10),
        # ragged: odd mesh, odd node count, odd velocity count
        march("cavity_51x45_p2_nc13", "cavity", 51, 45, 2, "nc13", "fp64", 10, kn=0.3),
        # the largest: the precision workload's mesh and velocities in FP64, and in FP32 storage
        march("cavity_128x128_p4_nc24", "cavity", 128, 128, 4, "nc24", "fp64", 2, kn=8.0),
        march("cavity_128x128_p4_nc24_fp32", "cavity", 128, 128, 4, "nc24", "fp32", 2, kn=8.0),
        # the headline problem in FP32 storage
        march("cavity_64x64_p3_nc16_fp32", "cavity", 64, 64, 3, "nc16", "fp32", 10),
        # a steady-state solve in the reference form: march, check the residual, fold, read the flow
        {"name": "steady_72x72_p2_nc16_ref", "kind": "steady", "flow": "cavity", "nx": 72, "ny": 72, "p": 2,
         "vel": "nc16", "precision": "fp32_ref", "steps": 25, "graph": 0, "kn": 1.0},
        # problems of the mixed batch's distribution advanced together
        {"name": "batch_10_fp64", "kind": "batch", "members": 10, "nlo": 16, "nhi": 64, "plo": 2, "phi": 4,
         "mlo": 8, "mhi": 16, "precision": "fp64", "steps": 5, "graph": 5, "shape_seed": 18},
        # the implicit marching of the flow's published runs, at ten explicit steps
        {"name": "implicit_32x32_p3_nc12", "kind": "implicit", "flow": "cavity", "nx": 32, "ny": 32, "p": 3,
         "vel": "nc12", "scheme": "backward_euler", "times_dt": 10.0, "kn": 1.0},
        # a set of small requests served together
        {"name": "serve_8_ref", "kind": "serve", "members": 8, "nlo": 16, "nhi": 28, "plo": 2, "phi": 3,
         "mlo": 6, "mhi": 12, "precision": "fp32_ref", "steps": 100, "check": 50, "shape_seed": 15},
    ]


def log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["march"] * 7 + ["steady"] * 2 + ["batch", "implicit"])
    if kind == "batch":
        return {"kind": "batch", "members": rng.randint(4, 10), "nlo": 16, "nhi": 64, "plo": 2, "phi": 4,
                "mlo": 8, "mhi": 16, "precision": rng.choice(["fp64", "fp32_ref"]), "steps": 5, "graph": 5,
                "shape_seed": rng.randrange(1 << 20)}
    while True:
        n = log_int(rng, 8, 128)
        c = {"kind": kind, "flow": rng.choice(["couette", "cavity"]), "nx": n,
             "ny": min(128, max(8, int(n * rng.uniform(0.75, 1.33)))), "p": rng.randint(1, 4),
             "vel": "gh4" if rng.random() < 0.3 else "nc%d" % rng.randint(6, 24),
             "kn": round(10.0 ** rng.uniform(-1.0, 1.0), 3)}
        if kind == "implicit":
            c.update(scheme=rng.choice(["backward_euler", "sdirk2"]), times_dt=float(rng.randint(4, 12)))
            if dof_of(c) <= 4_000_000:
                return c
            continue
        c.update(precision=rng.choice(["fp64", "fp64", "fp32", "fp32_ref"]), graph=rng.choice([0, 0, 5]))
        if kind == "steady":
            c["precision"] = rng.choice(["fp64", "fp32_ref"])
        c["steps"] = max(2, min(20, int(4e8 / dof_of(c))))
        if dof_of(c) * c["steps"] <= 4.7e8:
            return c


# ---- sizes --------------------------------------------------------------------------------------

def velocities(vel):
    n = int(vel[2:])
    return n * n


def dof_of(c):
    return c["nx"] * c["ny"] * (c["p"] + 1) ** 2 * velocities(c["vel"])


def members_of(c):
    """The problems of a batch or of a served set: shapes from the case alone."""
    rng = random.Random(c["shape_seed"])
    out = []
    for _ in range(c["members"]):
        n = rng.randint(c["nlo"], c["nhi"])
        out.append({"flow": rng.choice(["couette", "cavity"]), "nx": n, "ny": n,
                    "p": rng.randint(c["plo"], c["phi"]),
                    "vel": rng.choice(["gh4", "nc%d" % rng.randint(c["mlo"], c["mhi"])]),
                    "kn": 10.0 ** rng.uniform(-1.0, 1.0), "precision": c["precision"]})
    return out


def stage_work(c):
    """Bytes and operations of one evaluation of the right-hand side folded into an RK stage: the
    state read once and the new one written once; two derivative lines, two lifts, the collision, the
    three moments and the update for every value."""
    size = 8 if c.get("precision", "fp64") == "fp64" else 4
    n = dof_of(c)
    return 2.0 * size * n, n * (4.0 * (c["p"] + 1) + 4.0 + 14.0 + 6.0 + 4.0)


def work(case):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        parts = [stage_work(m) for m in members_of(case)]
        scale = 4.0 * case["steps"]
        return {"bytes": scale * sum(b for b, _ in parts), "flops": scale * sum(f for _, f in parts)}
    b, f = stage_work(case)
    if kind == "implicit":  # the state read and written once, and one evaluation a stage
        stages = 2 if case["scheme"] == "sdirk2" else 1
        return {"bytes": stages * b, "flops": stages * f}
    extra = 1 if kind == "steady" else 0  # the residual's evaluation
    return {"bytes": (4.0 * case["steps"] + extra) * b, "flops": (4.0 * case["steps"] + extra) * f}


# ---- preparing and running ------------------------------------------------------------------------

def velset(vel):
    return ("gh", int(vel[2:])) if vel.startswith("gh") else ("nc", int(vel[2:]), NC_VMAX)


def walls(flow, speed=LID):
    if flow == "couette":  # periodic in x, plates y = 0 and y = 1 moving in opposite directions
        return (1, 0, 1, 0), ((-speed, 0.0), (0.0, 0.0), (speed, 0.0), (0.0, 0.0))
    return (1, 1, 1, 1), ((0.0, 0.0), (0.0, 0.0), (speed, 0.0), (0.0, 0.0))


def fields(seed, x, y):
    """Smooth density and velocity fields at points x, y (numpy, 64 bits): four seeded modes each."""
    rng = np.random.default_rng(seed)
    out = []
    for base, amp in ((1.0, 0.02), (0.0, 0.03), (0.0, 0.03)):
        v = np.full_like(x, base)
        for _ in range(4):
            kx, ky = rng.integers(0, 4, 2)
            v = v + amp * rng.uniform(-1.0, 1.0) * np.cos(2 * np.pi * (kx * x + ky * y) + rng.uniform(0, 2 * np.pi))
        out.append(v)
    return out


def make_solver(c, seed):
    bc, wall_u = walls(c["flow"])
    s = dg.Solver(c["nx"], c["ny"], c["p"], velset(c["vel"]), dg.tau_from_kn(c["kn"]), bc, wall_u,
                  stream="torch", torch_memory=True, precision=c.get("precision", "fp64"))
    x, y = s.node_coords()
    s.init_moments(*fields(seed, x, y))
    return s


class DeviceView:
    """The current state on the device, f[element][velocity][node], as torch takes it without a copy;
    a tensor made of it keeps the solver, whose memory it is."""

    def __init__(self, solver, precision):
        self.solver = solver
        kind = "<f8" if precision == "fp64" else "<f4"
        self.__cuda_array_interface__ = {"shape": (solver.K, solver.Q, solver.Np), "typestr": kind,
                                         "data": (solver.state_device_ptr(), False), "version": 2}


def state_of(solver, precision):
    return torch.as_tensor(DeviceView(solver, precision), device="cuda")


def request_spec(m, seed):
    """A request: the member's problem with a seeded wall speed."""
    bc, wall_u = walls(m["flow"], LID * random.Random(seed).uniform(0.5, 1.5))
    return types.SimpleNamespace(nx=m["nx"], ny=m["ny"], p=m["p"], velset=velset(m["vel"]), tau=None, kn=m["kn"],
                                 kn_length=1.0, kn_convention=1, bc=bc, wall_u=wall_u, x0=0.0, y0=0.0,
                                 lx=1.0, ly=1.0)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        specs = [request_spec(m, seed * 1000 + i) for i, m in enumerate(members_of(case))]
        return {"case": case, "specs": specs}
    if kind == "batch":
        members = members_of(case)
        solvers = [make_solver(m, seed * 1000 + i) for i, m in enumerate(members)]
        return {"case": case, "solvers": solvers, "dt": [s.stable_dt(CFL) for s in solvers],
                "batch": dg.Batch(solvers, graph=case["graph"])}
    s = make_solver(case, seed)
    if case.get("graph"):
        s.set_graph(case["graph"])
    return {"case": case, "solver": s, "dt": s.stable_dt(CFL)}


def in_storage(precision, v):
    """Host results of the FP32 storage forms carry single precision."""
    return np.float64(v) if precision == "fp64" else np.float32(v)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "march":
        s = state["solver"]
        s.step(case["steps"], state["dt"])
        return state_of(s, case["precision"])
    if kind == "steady":
        s, prec = state["solver"], case["precision"]
        s.step(case["steps"], state["dt"])
        r = s.residual()
        if prec == "fp32_ref":
            s.fold()
        rho, ux, uy = s.moments()
        return {"residual": in_storage(prec, r), "rho": in_storage(prec, rho), "u": in_storage(prec, [ux, uy])}
    if kind == "batch":
        state["batch"].step(case["steps"], state["dt"])
        return {"residuals": in_storage(case["precision"], state["batch"].residuals()),
                "states": [state_of(s, case["precision"]) for s in state["solvers"]]}
    if kind == "implicit":
        s = state["solver"]
        s.implicit_step(1, case["times_dt"] * state["dt"], case["scheme"])
        return state_of(s, "fp64")
    server = dg.Server(64 << 30, max_active=16, precision=case["precision"], residual_target=1e-6,
                       check_every=case["check"], max_steps=case["steps"], cfl=CFL)
    ids = [server.submit(spec, 0.0) for spec in state["specs"]]
    server.run()
    out = []
    for i in ids:
        rho, ux, uy = server.moments(i)
        out.append([in_storage(case["precision"], rho), in_storage(case["precision"], [ux, uy])])
    server.close()
    return out


# ---- the same passes in plain torch, 64 bits --------------------------------------------------------

class Exact:
    """The semi-discrete system on arrays f[ny][nx][q][j][i] (j, i: nodes along y, x)."""

    def __init__(self, c, speed=LID):
        self.nx, self.ny, p = c["nx"], c["ny"], c["p"]
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        t = lambda a: torch.tensor(np.asarray(a), dtype=torch.float64, device=self.dev)  # noqa: E731
        # Gauss-Lobatto nodes, Legendre Vandermonde matrix, derivative, lifts
        leg = np.polynomial.legendre
        inner = leg.legroots(leg.legder([0.0] * p + [1.0])) if p > 1 else np.zeros(0)
        r = np.concatenate([[-1.0], np.sort(inner.real), [1.0]])
        V = leg.legvander(r, p) * np.sqrt(np.arange(p + 1) + 0.5)
        Vd = np.stack([leg.legval(r, leg.legder(np.eye(p + 1)[k])) * math.sqrt(k + 0.5) for k in range(p + 1)], 1)
        D, Minv = Vd @ np.linalg.inv(V), V @ V.T
        self.D, self.lo, self.hi = t(D), t(Minv[:, 0]), t(Minv[:, -1])
        hx, hy = 1.0 / self.nx, 1.0 / self.ny
        self.rx, self.sy = 2.0 / hx, 2.0 / hy
        # velocities
        n = int(c["vel"][2:])
        if c["vel"].startswith("gh"):
            x1, w1 = np.polynomial.hermite_e.hermegauss(n)
            w1 = w1 / w1.sum()
        else:
            x1 = np.linspace(-NC_VMAX, NC_VMAX, n)
            w1 = np.exp(-0.5 * x1 * x1)
            w1[0] *= 0.5
            w1[-1] *= 0.5
            w1 = w1 / w1.sum()
        ex, ey = np.tile(x1, n), np.repeat(x1, n)
        w = np.tile(w1, n) * np.repeat(w1, n)
        theta = 1.0 if c["vel"].startswith("gh") else float((w * ex * ex).sum())
        q = (1, 1, -1, 1, 1)
        self.ex, self.ey, self.w, self.theta = t(ex).view(q), t(ey).view(q), t(w).view(q), theta
        self.tau = c["kn"] / math.sqrt(math.pi / 2.0)
        self.dt = CFL * 0.5 * min(hx, hy) * float(np.min(np.diff(r))) / float(np.max(abs(ex) + abs(ey)))
        self.X = (np.arange(self.nx)[None, :, None, None] + 0.5 * (1 + r[None, None, None, :])) * hx
        self.Y = (np.arange(self.ny)[:, None, None, None] + 0.5 * (1 + r[None, None, :, None])) * hy
        self.X, self.Y = (np.broadcast_to(v, (self.ny, self.nx, p + 1, p + 1)) for v in (self.X, self.Y))
        self.shape = (self.ny, self.nx, len(w), p + 1, p + 1)
        self.t = t
        # walls: the exterior equilibrium over its incoming flux, per side (bottom, right, top, left)
        bc, wall_u = walls(c["flow"], speed)
        self.wall = [None] * 4
        for side, en in enumerate((-self.ey, self.ex, self.ey, -self.ex)):
            if bc[side]:
                g = self.equilibrium(torch.ones(1, 1, 1, 1, 1, dtype=torch.float64, device=self.dev), *wall_u[side])
                self.wall[side] = (g / (torch.clamp(-en, min=0.0) * g).sum(), torch.clamp(en, min=0.0))
        self.scale = 1.0 / speed

    def equilibrium(self, rho, ux, uy):
        eu = self.ex * ux + self.ey * uy
        return self.w * rho * (1.0 + eu / self.theta + eu * eu / (2.0 * self.theta ** 2)
                               - (ux * ux + uy * uy) / (2.0 * self.theta))

    def start(self, seed):
        rho, ux, uy = (self.t(v).unsqueeze(2) for v in fields(seed, self.X, self.Y))
        return self.equilibrium(rho, ux, uy)

    def rest(self):
        return self.equilibrium(torch.ones(self.ny, self.nx, 1, *self.shape[3:], dtype=torch.float64, device=self.dev),
                                0.0, 0.0)

    def sums(self, f):
        return f.sum(2, keepdim=True), (self.ex * f).sum(2, keepdim=True), (self.ey * f).sum(2, keepdim=True)

    def flow(self, f):
        rho, mx, my = self.sums(f)
        return rho, mx / rho, my / rho

    def outside(self, own, other, side, axis, at):
        """The exterior trace of a side: the neighbour's, or the wall's diffuse reflection."""
        if self.wall[side] is None:
            return other
        g, out = self.wall[side]
        g, out = g.squeeze(-1), out.squeeze(-1)
        edge = own.narrow(axis, at, 1)
        other = other.clone()
        other.narrow(axis, at, 1).copy_((out * edge).sum(2, keepdim=True) * g)
        return other

    def rate(self, f):
        k = torch.matmul(f, self.D.T).mul_(-self.rx * self.ex)
        k.sub_(torch.matmul(self.D, f).mul_(self.sy * self.ey))
        ex, ey = self.ex.squeeze(-1), self.ey.squeeze(-1)
        left, right, bottom, top = f[..., 0], f[..., -1], f[..., 0, :], f[..., -1, :]
        nx, ny = self.nx, self.ny
        J = torch.clamp(ex, min=0.0) * (left - self.outside(left, right.roll(1, 1), 3, 1, 0)) * self.rx
        k.sub_(J.unsqueeze(-1) * self.lo)
        J = torch.clamp(-ex, min=0.0) * (right - self.outside(right, left.roll(-1, 1), 1, 1, nx - 1)) * self.rx
        k.sub_(J.unsqueeze(-1) * self.hi)
        J = torch.clamp(ey, min=0.0) * (bottom - self.outside(bottom, top.roll(1, 0), 0, 0, 0)) * self.sy
        k.sub_(J.unsqueeze(-2) * self.lo.view(-1, 1))
        J = torch.clamp(-ey, min=0.0) * (top - self.outside(top, bottom.roll(-1, 0), 2, 0, ny - 1)) * self.sy
        k.sub_(J.unsqueeze(-2) * self.hi.view(-1, 1))
        return k.add_((self.equilibrium(*self.flow(f)) - f).div_(self.tau))

    def march(self, f, steps):
        dt = self.dt
        for _ in range(steps):
            k = self.rate(f)
            total = k.clone()
            for a, b in ((0.5, 2.0), (0.5, 2.0), (1.0, 1.0)):
                k = self.rate(f + a * dt * k)
                total.add_(k, alpha=b)
            f = f.add(total, alpha=dt / 6.0)
        return f

    def residual(self, f):
        return max(float(s.abs().max()) for s in self.sums(self.rate(f))) * self.scale

    def solve(self, b, h):
        """y - h L(y) = b: Newton's method with GMRES(40), products by forward differentiation."""
        y = b.clone()
        first = None
        for _ in range(12):
            F = b - y + h * self.rate(y)
            size = float(F.norm())
            first = first or size
            if size <= 1e-13 * first:
                break
            # one GMRES cycle for (I - h J) d = F
            basis, H = [F / size], np.zeros((41, 40))
            for j in range(40):
                v = basis[j]
                z = v - h * torch.func.jvp(self.rate_pure, (y,), (v,))[1]
                for _pass in range(2):
                    for i, u in enumerate(basis):
                        c = float((u * z).sum())
                        H[i, j] += c
                        z = z - c * u
                H[j + 1, j] = float(z.norm())
                e = np.zeros(j + 2)
                e[0] = size
                s = np.linalg.lstsq(H[:j + 2, :j + 1], e, rcond=None)[0]
                if np.linalg.norm(e - H[:j + 2, :j + 1] @ s) <= 1e-8 * size or H[j + 1, j] <= 1e-30:
                    break
                basis.append(z / H[j + 1, j])
            for i, c in enumerate(s):
                y = y + float(c) * basis[i]
        return y

    def rate_pure(self, f):
        """rate() without updates in place, for differentiation."""
        ex, ey = self.ex.squeeze(-1), self.ey.squeeze(-1)
        k = -self.rx * self.ex * torch.matmul(f, self.D.T) - self.sy * self.ey * torch.matmul(self.D, f)
        traces = ((f[..., 0], f[..., -1].roll(1, 1), 3, 1, 0, ex, self.rx, self.lo, -1),
                  (f[..., -1], f[..., 0].roll(-1, 1), 1, 1, self.nx - 1, -ex, self.rx, self.hi, -1),
                  (f[..., 0, :], f[..., -1, :].roll(1, 0), 0, 0, 0, ey, self.sy, self.lo, -2),
                  (f[..., -1, :], f[..., 0, :].roll(-1, 0), 2, 0, self.ny - 1, -ey, self.sy, self.hi, -2))
        for own, other, side, axis, at, en, scale, lift, dim in traces:
            if self.wall[side] is not None:
                g, out = (v.squeeze(-1) for v in self.wall[side])
                diffuse = (out * own).sum(2, keepdim=True) * g
                on = torch.zeros(own.shape[axis], dtype=torch.bool, device=own.device)
                on[at] = True
                other = torch.where(on.view([-1 if a == axis else 1 for a in range(own.dim())]), diffuse, other)
            J = torch.clamp(en, min=0.0) * (own - other) * scale
            k = k - J.unsqueeze(dim) * (lift if dim == -1 else lift.view(-1, 1))
        return k + (self.equilibrium(*self.flow(f)) - f) / self.tau


def as_state(f):
    ny, nx, q, n1, _ = f.shape
    return f.reshape(ny * nx, q, n1 * n1)


def as_nodes(v):
    return v.reshape(v.shape[0] * v.shape[1], -1)


def deviation(e, f, f0, precision):
    """What the state array of a precision holds of f: all of it, the deviation from rest, or from the
    reference."""
    if precision == "fp64":
        return f
    return f - e.w if precision == "fp32" else f - f0


def exact(case, seed):
    kind = case["kind"]
    if kind == "serve":
        out = []
        for i, m in enumerate(members_of(case)):
            e = Exact(m, LID * random.Random(seed * 1000 + i).uniform(0.5, 1.5))
            rho, ux, uy = (as_nodes(v).reshape(-1) for v in e.flow(e.march(e.rest(), case["steps"])))
            out.append([rho, torch.stack([ux, uy])])
        return out
    if kind == "batch":
        residuals, states = [], []
        for i, m in enumerate(members_of(case)):
            e = Exact(m)
            f0 = e.start(seed * 1000 + i)
            f = e.march(f0, case["steps"])
            residuals.append(e.residual(f))
            states.append(as_state(deviation(e, f, f0, case["precision"])))
        return {"residuals": np.array(residuals), "states": states}
    e = Exact(case)
    f0 = e.start(seed)
    if kind == "implicit":
        if dof_of(case) > 4_000_000:
            return None
        h, f = case["times_dt"] * e.dt, f0
        if case["scheme"] == "backward_euler":
            return as_state(e.solve(f, h))
        g = 1.0 - math.sqrt(0.5)  # Alexander's two stages
        y = e.solve(f, g * h)
        return as_state(e.solve(f + (1.0 - g) * h * e.rate(y), g * h))
    f = e.march(f0, case["steps"])
    if kind == "steady":
        rho, ux, uy = (as_nodes(v) for v in e.flow(f))
        return {"residual": np.float64(e.residual(f)), "rho": rho, "u": torch.stack([ux, uy])}
    return as_state(deviation(e, f, f0, case["precision"]))
