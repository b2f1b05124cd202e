"""The work that users of this framework have it do, as cases that can be timed.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare`` builds what a program holds before the call (solver, batch,
network, inputs made from the seed on the GPU), ``run`` makes one pass through
the public entry points, ``work`` says what the pass cannot do without, and
``exact`` gives the results in 64 bits by plain torch, without the library.

Kinds of work:
  step2d   time steps of one 2D grid on the fused path: a periodic vortex, an
           inlet channel (inflow, slip walls, outflow), a closed viscous box, a
           ramp inlet on a curvilinear grid
  step3d   time steps of one 3D grid on the fused path: a tilted Sod tube or a
           channel with walls and an inflow face
  batch    time steps of many uneven 2D grids together
  split    time steps on the tunable path, the library's default, and the
           residual that a convergence monitor looks at
  rollout  a differentiable rollout: forward steps, an objective, its gradient
  train    the tuner's network: epochs of minibatch training, then prediction
  sweep    the tuner's prediction of a launch space and its best entries
"""
import math
import random

import numpy as np
import torch

from paper_2306_14011_amd import autotune, fv, inputs, rollout, tune_space

GAMMA = 1.4
DEV = "cuda"

PERIODIC, OUTFLOW, WALL, INFLOW = 0, 1, 2, 3


def listed():
    return [
        # the smallest grid in use: every launch counts
        {"name": "step2d-64", "kind": "step2d", "flow": "vortex", "nx": 64, "ny": 64, "scheme": "minmod",
         "source": False, "steps": 16},
        # an ordinary channel flow, ragged sizes, every kind of boundary
        {"name": "step2d-channel-403x277", "kind": "step2d", "flow": "channel", "nx": 403, "ny": 277,
         "scheme": "vanleer", "source": False, "steps": 8},
        # the benchmark's grid
        {"name": "step2d-2048", "kind": "step2d", "flow": "vortex", "nx": 2048, "ny": 2048, "scheme": "minmod",
         "source": False, "steps": 8},
        # Navier-Stokes in a closed box
        {"name": "step2d-viscous-1024", "kind": "step2d", "flow": "box", "nx": 1024, "ny": 1024, "scheme": "minmod",
         "source": False, "steps": 6},
        # a supersonic inlet with a ramp on a curvilinear grid of the paper's size
        {"name": "step2d-ramp-3328x1024", "kind": "step2d", "flow": "ramp", "nx": 3328, "ny": 1024,
         "scheme": "minmod", "source": False, "steps": 4},
        # the benchmark's 3D workload
        {"name": "step3d-sod-256", "kind": "step3d", "flow": "sod", "nx": 256, "ny": 256, "nz": 256,
         "scheme": "minmod", "source": False, "steps": 2},
        # a small 3D channel, ragged sizes, walls and inflow
        {"name": "step3d-channel-97x61x45", "kind": "step3d", "flow": "channel", "nx": 97, "ny": 61, "nz": 45,
         "scheme": "minmod", "source": False, "steps": 4},
        # a parameter study: 96 uneven grids together, more than the caches hold
        {"name": "batch-96", "kind": "batch", "count": 96, "smin": 128, "smax": 1024, "scheme": "minmod", "steps": 8},
        # the path a solver starts on, and the residual of its convergence monitor
        {"name": "split-1024", "kind": "split", "ndim": 2, "nx": 1024, "ny": 1024, "nz": 1, "scheme": "minmod",
         "steps": 2},
        # the gradient of an objective through 20 steps, checkpoints every 10
        {"name": "rollout-512", "kind": "rollout", "nx": 512, "ny": 512, "scheme": "minmod", "steps": 20, "every": 10},
        # training on the 3D tuner's 1500 rows, two epochs, and the test rows' prediction
        {"name": "train-1500", "kind": "train", "rows": 1500, "epochs": 2, "test": 500, "n_in": 14},
        # the whole 2D launch space
        {"name": "sweep-2d", "kind": "sweep", "begin": 0, "count": 189062500, "k": 8, "n_in": 14},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["step2d", "step2d", "step2d", "step3d", "step3d", "batch", "split", "rollout", "train", "sweep"])
    if kind == "step2d":
        flow = rng.choice(["vortex", "vortex", "channel", "box", "ramp"])
        nx, ny = _log(rng, 48, 2048), _log(rng, 48, 2048)
        scheme = rng.choice(["minmod", "vanleer"] + (["kappa-1", "kappa1/3"] if flow == "vortex" else []))
        return {"kind": kind, "flow": flow, "nx": nx, "ny": ny, "scheme": scheme,
                "source": flow == "vortex" and rng.random() < 0.25, "steps": rng.randint(4, 8)}
    if kind == "step3d":
        flow = rng.choice(["sod", "channel"])
        return {"kind": kind, "flow": flow, "nx": _log(rng, 24, 256), "ny": _log(rng, 24, 256),
                "nz": _log(rng, 24, 256), "scheme": rng.choice(["minmod", "vanleer"]),
                "source": False, "steps": rng.randint(1, 2)}
    if kind == "batch":
        smin = _log(rng, 48, 256)
        return {"kind": kind, "count": rng.randint(3, 96), "smin": smin, "smax": rng.randint(smin, 4 * smin),
                "scheme": rng.choice(["minmod", "vanleer"]), "steps": rng.randint(4, 8)}
    if kind == "split":
        if rng.random() < 0.5:
            return {"kind": kind, "ndim": 2, "nx": _log(rng, 64, 2048), "ny": _log(rng, 64, 2048), "nz": 1,
                    "scheme": rng.choice(["minmod", "vanleer"]), "steps": rng.randint(1, 3)}
        return {"kind": kind, "ndim": 3, "nx": _log(rng, 24, 192), "ny": _log(rng, 24, 192), "nz": _log(rng, 24, 192),
                "scheme": rng.choice(["minmod", "vanleer"]), "steps": rng.randint(1, 2)}
    if kind == "rollout":
        return {"kind": kind, "nx": _log(rng, 64, 640), "ny": _log(rng, 64, 640), "scheme": "minmod",
                "steps": rng.randint(6, 20), "every": rng.randint(3, 10)}
    if kind == "train":
        return {"kind": kind, "rows": _log(rng, 100, 1500), "epochs": rng.randint(1, 2),
                "test": _log(rng, 40, 2500), "n_in": rng.choice([14, 16])}
    space = 189062500
    count = _log(rng, 100000, space)
    return {"kind": kind, "begin": rng.randint(0, space - count), "count": count, "k": rng.randint(1, 8),
            "n_in": rng.choice([14, 16])}


# ---------------------------------------------------------------------------
# Flows: a plain description of the grid and its initial state.

class Flow:
    """Grid, boundary kinds and initial state of one flow (plain values and
    GPU tensors made from the seed)."""

    def __init__(self, case, seed):
        self.rng = np.random.default_rng(seed)
        self.case = case
        self.ndim = 3 if case["kind"] == "step3d" or case.get("ndim") == 3 else 2
        self.n = (case["nx"], case["ny"], case["nz"] if self.ndim == 3 else 1)
        self.lo, self.hi = (0.0, 0.0, 0.0), (1.0, 1.0, 1.0)
        self.bc = ((PERIODIC, PERIODIC),) * 3
        self.cfl = 0.5
        self.mu, self.prandtl = 0.0, 0.72
        self.bc_state = None
        self.nodes = None
        self.source = None
        self.scheme = case["scheme"]
        flow = case.get("flow") or {"split": "vortex" if self.ndim == 2 else "sod", "rollout": "sines"}[case["kind"]]
        getattr(self, "_" + flow)()
        if case.get("source"):
            self.source = 0.05 * self._modes(self.ndim + 2)

    # cell centres, broadcastable against (nz, ny, nx)
    def _axes(self):
        out = []
        for d in range(3):
            h = (self.hi[d] - self.lo[d]) / self.n[d]
            c = self.lo[d] + h * (torch.arange(self.n[d], dtype=torch.float64, device=DEV) + 0.5)
            out.append(c.view([-1 if a == 2 - d else 1 for a in range(3)]))
        return out

    # `count` smooth periodic fields, three sine modes each
    def _modes(self, count):
        x, y, z = self._axes()
        f = torch.zeros((count, self.n[2], self.n[1], self.n[0]), dtype=torch.float64, device=DEV)
        L = [self.hi[d] - self.lo[d] for d in range(3)]
        for v in range(count):
            for _ in range(3):
                k = self.rng.integers(1, 4, 3)
                a = 2 * math.pi * (float(k[0]) * (x - self.lo[0]) / L[0] + float(k[1]) * (y - self.lo[1]) / L[1])
                if self.ndim == 3:
                    a = a + 2 * math.pi * float(k[2]) * (z - self.lo[2]) / L[2]
                f[v] += torch.sin(a + float(self.rng.uniform(0, 2 * math.pi)))
        return f

    def _pack(self, rho, vel, p):
        U = torch.zeros((self.ndim + 2, self.n[2], self.n[1], self.n[0]), dtype=torch.float64, device=DEV)
        U[0] = rho
        ke = 0.0
        for d in range(self.ndim):
            U[1 + d] = rho * vel[d]
            ke = ke + vel[d] * vel[d]
        U[self.ndim + 1] = p / (GAMMA - 1.0) + 0.5 * rho * ke
        self.U = U

    def _bumps(self, count, sigma, amp):
        x, y, _ = self._axes()
        f = 0.0
        L = [self.hi[d] - self.lo[d] for d in range(2)]
        for _ in range(count):
            c = [float(self.rng.uniform(self.lo[d], self.hi[d])) for d in range(2)]
            # the product of two 1D bumps
            gx = torch.exp(-((x - c[0]) / (sigma * L[0])) ** 2 / 2)
            gy = torch.exp(-((y - c[1]) / (sigma * L[1])) ** 2 / 2)
            f = f + amp * gx * gy
        return f

    def _vortex(self):
        # isentropic vortex on a Mach 0.5 diagonal stream with 32 density bumps
        self.hi = (10.0, 10.0, 1.0)
        x, y, _ = self._axes()
        c = 5.0 + self.rng.uniform(-0.5, 0.5, 2)
        beta = 5.0
        s = 0.5 * math.sqrt(GAMMA / 2)
        dx, dy = x - float(c[0]), y - float(c[1])
        dx = dx - 10.0 * torch.round(dx / 10.0)
        dy = dy - 10.0 * torch.round(dy / 10.0)
        f = torch.exp(0.5 * (1.0 - dx * dx - dy * dy))
        u = s - beta / (2 * math.pi) * f * dy
        v = s + beta / (2 * math.pi) * f * dx
        T = 1.0 - (GAMMA - 1.0) * beta * beta / (8 * GAMMA * math.pi ** 2) * f * f
        rho = T ** (1.0 / (GAMMA - 1.0))
        p = rho * T
        self._pack(rho + self._bumps(32, 0.025, 1e-2), (u, v), p)

    def _inflow_state(self, mach, angle):
        c = math.sqrt(GAMMA)
        vel = [mach * c * math.cos(angle), mach * c * math.sin(angle), 0.0][: self.ndim]
        q = [1.0] + vel + [1.0 / (GAMMA - 1.0) + 0.5 * sum(a * a for a in vel)]
        self.bc_state = np.zeros((3, 2, 5))
        self.bc_state[0, 0, : len(q)] = q
        return vel

    def _channel(self):
        # supersonic inflow at a small angle, slip walls, outflow; in 3D periodic along z
        self.hi = (2.0, 1.0, 1.0)
        self.bc = ((INFLOW, OUTFLOW), (WALL, WALL), (PERIODIC, PERIODIC))
        vel = self._inflow_state(2.0, 0.05)
        rho = 1.0 + self._bumps(12, 0.08, 0.02)
        p = 1.0 + self._bumps(12, 0.08, 0.02)
        if self.ndim == 3:
            _, _, z = self._axes()
            rho = rho * (1.0 + 0.02 * torch.sin(2 * math.pi * z))
        self._pack(rho, vel, p)

    def _box(self):
        # a pressure pulse in a closed box, Navier-Stokes
        self.bc = ((WALL, WALL), (WALL, WALL), (PERIODIC, PERIODIC))
        self.mu = 1e-4
        x, y, _ = self._axes()
        a = [float(t) for t in self.rng.uniform(0.05, 0.2, 3)]
        u = a[0] * torch.sin(math.pi * x) * torch.cos(math.pi * y)
        v = a[1] * torch.cos(math.pi * x) * torch.sin(math.pi * y)
        self._pack(1.0 + self._bumps(6, 0.1, 0.05), (u, v), 1.0 + a[2] * torch.cos(math.pi * x) * torch.cos(math.pi * y))

    def _ramp(self):
        # Mach 2.5 inflow over a floor that turns up by 10 degrees, curvilinear grid
        self.hi = (3.0, 1.0, 1.0)
        self.bc = ((INFLOW, OUTFLOW), (WALL, OUTFLOW), (PERIODIC, PERIODIC))
        vel = self._inflow_state(2.5, 0.0)
        nx, ny, _ = self.n
        xi = 3.0 * np.arange(nx + 1) / nx
        # smoothed corner at x = 1
        w = 0.1
        floor = math.tan(math.radians(10.0)) * w * np.logaddexp(0.0, (xi - 1.0) / w)
        eta = np.arange(ny + 1) / ny
        yy = floor[None, :] + (1.0 + 0.0 * floor[None, :] - floor[None, :]) * eta[:, None]
        self.nodes = np.stack([np.broadcast_to(xi, yy.shape), yy])
        self._pack(1.0 + self._bumps(12, 0.08, 0.02), vel, 1.0 + self._bumps(12, 0.08, 0.02))

    def _sod(self):
        # a tilted shock tube: transmissive x, periodic y and z
        self.bc = ((OUTFLOW, OUTFLOW), (PERIODIC, PERIODIC), (PERIODIC, PERIODIC))
        th, ph = float(self.rng.uniform(0, math.pi / 6)), float(self.rng.uniform(0, 2 * math.pi))
        x, y, z = self._axes()
        s = (x - 0.5) * math.cos(th) + (y - 0.5) * math.sin(th) * math.cos(ph) + (z - 0.5) * math.sin(th) * math.sin(ph)
        left = s < 0
        one = torch.ones_like(s)
        self._pack(torch.where(left, one, 0.125 * one), (0.0, 0.0, 0.0), torch.where(left, one, 0.1 * one))

    def _sines(self):
        # smooth everywhere: no flat regions, where a limiter's derivative is undefined
        f = self._modes(4)
        self._pack(1.0 + 0.05 * f[0], (0.4 + 0.05 * f[1], 0.3 + 0.05 * f[2]), 1.0 + 0.05 * f[3])

    # -- the framework's description of the same grid
    def spec(self):
        s = inputs.GridSpec(self.ndim, tuple(int(v) for v in self.n), self.lo, self.hi, self.bc, GAMMA, self.cfl)
        if self.scheme == "vanleer":
            s.limiter = "vanleer"
        elif self.scheme.startswith("kappa"):
            s.limiter, s.kappa = False, {"kappa-1": -1.0, "kappa1/3": 1.0 / 3.0}[self.scheme]
        s.mu, s.prandtl, s.bc_state, s.nodes = self.mu, self.prandtl, self.bc_state, self.nodes
        return s


def _batch_grids(case, seed):
    """Sizes (from the case alone) and vortex parameters (from the seed)."""
    sizes = np.random.default_rng(case["count"] * 1000003 + case["smin"] * 1009 + case["smax"])
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(case["count"]):
        nx, ny = (int(v) for v in sizes.integers(case["smin"], case["smax"] + 1, 2))
        out.append((nx, ny, int(rng.integers(0, 1 << 30))))
    return out


def _train_data(case, seed):
    """Standardised launch features and a runtime that depends on them."""
    rng = np.random.default_rng(seed)
    n = case["rows"] + case["test"]
    X = rng.integers(0, 5, (n, case["n_in"])).astype(np.float64)
    y = ((X - rng.integers(0, 5, case["n_in"])) ** 2 * rng.uniform(0.01, 0.2, case["n_in"])).sum(1)
    y = np.log(1.0 + y) + 0.02 * rng.standard_normal(n)
    X = (X - X.mean(0)) / X.std(0)
    y = (y - y.mean()) / y.std()
    order = np.stack([rng.permutation(case["rows"]) for _ in range(case["epochs"])]).astype(np.int32)
    return X.astype(np.float32), y.astype(np.float32), order


def _space(case):
    """The 2D launch space with standardised features."""
    g = inputs.grid2d(2048, 2048)
    ls = tune_space.LaunchSpace.for_grid(g)
    F = ls.features(ls.sample(300, 0))
    extra = [0.3, -0.7] if case["n_in"] == 16 else []
    mean, std = F.mean(axis=0), F.std(axis=0)
    sp = ls.struct(mean, np.where(std == 0.0, 1.0, std))
    if extra:
        sp.n_extra = 2
        sp.extra[0], sp.extra[1] = extra
    return sp


# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind in ("step2d", "step3d", "split", "rollout"):
        f = Flow(case, seed)
        st["spec"] = f.spec()
        st["solver"] = fv.Solver(st["spec"], device=DEV)
        if kind != "split":
            st["solver"].set_path(fv.FV_PATH_FUSED)
        if f.source is not None:
            st["solver"].set_source(f.source)
        if kind == "rollout":
            st["U0"] = f.U.clone().requires_grad_(True)
        else:
            st["solver"].interior().copy_(f.U)
            st["dt"] = torch.zeros(case["steps"], dtype=torch.float64, device=DEV)
    elif kind == "batch":
        specs, states = [], []
        for nx, ny, s in _batch_grids(case, seed):
            f = Flow({"kind": "step2d", "flow": "vortex", "nx": nx, "ny": ny, "scheme": case["scheme"]}, s)
            specs.append(f.spec())
            states.append(f.U)
        st["batch"] = fv.Batch(specs, device=DEV)
        for g, U in enumerate(states):
            st["batch"].view(g).copy_(U)
    elif kind == "train":
        st["X"], st["y"], st["order"] = _train_data(case, seed)
        st["seed"] = seed
    else:
        st["space"] = _space(case)
        st["net"] = autotune.Network(seed, device=DEV, n_in=case["n_in"])
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("step2d", "step3d"):
        state["solver"].step(case["steps"], dt_out=state["dt"])
        return {"U": state["solver"].interior(), "dt": state["dt"]}
    if kind == "split":
        state["solver"].step(case["steps"], dt_out=state["dt"])
        return {"U": state["solver"].interior(), "dt": state["dt"], "R": state["solver"].residual()}
    if kind == "batch":
        b = state["batch"]
        b.step(case["steps"])
        return {"U": b.U}
    if kind == "rollout":
        U, dts = rollout.rollout(state["U0"], state["solver"], case["steps"], case["every"])
        m = min(case["nx"], case["ny"])
        obj = rollout.pressure_integral(U, state["spec"], (m // 2 - m // 16, m // 2 + m // 16))
        (grad,) = torch.autograd.grad(obj, state["U0"])
        return {"U": U.detach(), "dt": dts, "objective": obj.detach(), "grad": grad}
    if kind == "train":
        # a fresh network, as every fit of the tuner makes one
        n = case["rows"]
        net = autotune.Network(state["seed"], device=DEV, n_in=case["n_in"])
        losses = net.train(state["X"][:n], state["y"][:n], order=state["order"], max_epochs=case["epochs"])
        return {"params": net.params, "m": net.m, "v": net.v, "losses": losses, "pred": net.predict(state["X"][n:])}
    idx, val = state["net"].sweep(state["space"], case["begin"], case["count"], case["k"])
    return {"index": np.array(idx, dtype=np.int64), "value": np.array(val, dtype=np.float32)}


def work(case):
    kind = case["kind"]
    # a step reads the state and writes it (the stages' states need not leave the chip)
    stage2, stage3 = 350, 620  # operations of one Runge-Kutta stage per cell
    if kind == "train":
        rows = case["rows"] * case["epochs"]
        np_ = 64 * case["n_in"] + 8449
        return {"bytes": 4 * (rows * (case["n_in"] + 2) + case["test"] * (case["n_in"] + 1) + 8 * np_),
                "flops": 2 * np_ * (3 * rows + case["test"])}
    if kind == "sweep":
        return {"bytes": 4 * (64 * case["n_in"] + 8449), "flops": 2 * (64 * case["n_in"] + 8256) * case["count"]}
    if kind == "batch":
        cells = sum(nx * ny for nx, ny, _ in _batch_grids(case, 0))
        return {"bytes": 64 * cells * case["steps"], "flops": 3 * stage2 * cells * case["steps"]}
    cells = case["nx"] * case["ny"] * case.get("nz", 1)
    three = kind == "step3d" or case.get("ndim") == 3
    nv, per = (5, stage3) if three else (4, stage2)
    b, f = 16 * nv * cells * case["steps"], 3 * per * cells * case["steps"]
    if kind == "split":
        return {"bytes": b + 16 * nv * cells, "flops": f + per * cells}
    if kind == "rollout":
        # forward, the recomputation from checkpoints, the reverse of each stage
        return {"bytes": 4 * b, "flops": 2 * f + 3 * f}
    if case.get("flow") == "ramp":
        b += 56 * cells * case["steps"]
        f = int(1.2 * f)
    if case.get("flow") == "box":
        f = int(1.3 * f)
    if case.get("source"):
        b += 8 * nv * cells * case["steps"]
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# The same results in 64 bits, by plain torch.

def _take(U, idx, ax):
    """Cells idx along axis ax (0 x, 1 y, 2 z) of (nvar, nz, ny, nx)."""
    return U.index_select(3 - ax, torch.as_tensor(idx, device=U.device))


def _pad(f, U, ax, w=2, normals=None):
    """U with w ghost layers on both ends of axis ax. normals: unit normals of
    the low and high wall faces (curvilinear), each (2, cross-section)."""
    n = U.shape[3 - ax]
    parts = []
    for side in (0, 1):
        kind = f.bc[ax][side]
        gpos = list(range(-w, 0)) if side == 0 else list(range(n, n + w))
        if kind == PERIODIC:
            g = _take(U, [p % n for p in gpos], ax)
        elif kind == WALL:
            g = _take(U, [-1 - p if side == 0 else 2 * n - 1 - p for p in gpos], ax).clone()
            if normals is None:
                g[1 + ax] = -g[1 + ax]
            else:
                nx, ny = normals[side]
                mn = g[1] * nx + g[2] * ny
                g[1] = g[1] - 2 * mn * nx
                g[2] = g[2] - 2 * mn * ny
        else:
            g = _take(U, [0 if side == 0 else n - 1] * w, ax)
            if kind == INFLOW:
                q = torch.as_tensor(f.bc_state[ax][side][: U.shape[0]], device=U.device)
                g = q.view(-1, 1, 1, 1).expand_as(g)
        parts.append(g)
    return torch.cat([parts[0], U, parts[1]], dim=3 - ax)


def _slope(a, b, scheme):
    """Limited difference of a cell from its two differences; at a tie the
    derivative follows a."""
    zero = torch.zeros_like(a)
    if scheme == "vanleer":
        ab = a * b
        return torch.where(ab > 0, 2 * ab / torch.where(ab > 0, a + b, torch.ones_like(a)), zero)
    same = ((a > 0) & (b > 0)) | ((a < 0) & (b < 0))
    return torch.where(same, torch.where(a.abs() <= b.abs(), a, b), zero)


def _states(P, dim, n, scheme):
    """Left and right states of the n + 1 faces from the padded line P."""
    q = [P.narrow(dim, k, n + 1) for k in range(4)]
    dm, dc, dp = q[1] - q[0], q[2] - q[1], q[3] - q[2]
    if scheme.startswith("kappa"):
        k = {"kappa-1": -1.0, "kappa1/3": 1.0 / 3.0}[scheme]
        a, b = 0.25 * (1 - k), 0.25 * (1 + k)
        return q[1] + a * dm + b * dc, q[2] - b * dc - a * dp
    return q[1] + 0.5 * _slope(dm, dc, scheme), q[2] - 0.5 * _slope(dc, dp, scheme)


def _roe(L, R, ax, nd):
    g1 = GAMMA - 1.0

    def prim(q):
        u = [q[1 + d] / q[0] for d in range(nd)]
        p = g1 * (q[nd + 1] - 0.5 * q[0] * sum(a * a for a in u))
        return u, p, (q[nd + 1] + p) / q[0]

    uL, pL, HL = prim(L)
    uR, pR, HR = prim(R)
    sL, sR = torch.sqrt(L[0]), torch.sqrt(R[0])
    w = sL / (sL + sR)
    ut = [w * a + (1 - w) * b for a, b in zip(uL, uR)]
    H = w * HL + (1 - w) * HR
    rt = sL * sR
    qq = sum(a * a for a in ut)
    c2 = g1 * (H - 0.5 * qq)
    c = torch.sqrt(c2)
    un = ut[ax]
    dp, dun, dr = pR - pL, uR[ax] - uL[ax], R[0] - L[0]
    w1 = (un - c).abs() * (dp - rt * c * dun) / (2 * c2)
    w2 = un.abs() * (dr - dp / c2)
    w5 = (un + c).abs() * (dp + rt * c * dun) / (2 * c2)
    ws = un.abs() * rt
    D = [w1 + w2 + w5]
    De = w1 * (H - un * c) + w2 * 0.5 * qq + w5 * (H + un * c)
    for d in range(nd):
        if d == ax:
            D.append(w1 * (un - c) + w2 * un + w5 * (un + c))
        else:
            du = uR[d] - uL[d]
            D.append((w1 + w2 + w5) * ut[d] + ws * du)
            De = De + ws * du * ut[d]
    D.append(De)
    F = []
    for v in range(nd + 2):
        fl, fr = L[v] * uL[ax], R[v] * uR[ax]
        if v == 1 + ax:
            fl, fr = fl + pL, fr + pR
        if v == nd + 1:
            fl, fr = (L[v] + pL) * uL[ax], (R[v] + pR) * uR[ax]
        F.append(0.5 * (fl + fr - D[v]))
    return torch.stack(F)


def _viscous(f, U, ax):
    """F_nu,n on the faces of axis ax (2D)."""
    P = _pad(f, _pad(f, U, 1, 1), 0, 1)[:, 0]  # (4, ny + 2, nx + 2)
    u, v = P[1] / P[0], P[2] / P[0]
    T = (GAMMA - 1) * (P[3] - 0.5 * P[0] * (u * u + v * v)) / P[0]
    w = torch.stack([u, v, T])
    h = [(f.hi[d] - f.lo[d]) / f.n[d] for d in range(2)]
    if ax == 1:
        w = w.transpose(1, 2)
    # faces between neighbours along the last axis; tangential along the middle one
    a, b = w[:, :, :-1], w[:, :, 1:]
    gn = ((b - a) / h[ax])[:, 1:-1]
    t = ((a[:, 2:] - a[:, :-2]) + (b[:, 2:] - b[:, :-2])) / (4 * h[1 - ax])
    gx, gy = (gn, t) if ax == 0 else (t, gn)
    div = gx[0] + gy[1]
    txx, tyy, txy = f.mu * (2 * gx[0] - 2 / 3 * div), f.mu * (2 * gy[1] - 2 / 3 * div), f.mu * (gx[1] + gy[0])
    t0, t1 = (txx, txy) if ax == 0 else (txy, tyy)
    um = 0.5 * (a + b)[:, 1:-1]
    k = f.mu * GAMMA / ((GAMMA - 1) * f.prandtl)
    out = torch.stack([torch.zeros_like(t0), t0, t1, um[0] * t0 + um[1] * t1 + k * gn[2]])
    out = out if ax == 0 else out.transpose(1, 2)
    return out[:, None]


class _Metrics:
    """Face normals, lengths and cell areas of a node array."""

    def __init__(self, nodes):
        X, Y = (torch.as_tensor(np.ascontiguousarray(a), device=DEV) for a in nodes)
        self.n, self.len = [], []
        for ax in (0, 1):
            if ax == 0:
                ex, ey = X[1:] - X[:-1], Y[1:] - Y[:-1]
                s = (ey, -ex)
            else:
                ex, ey = X[:, 1:] - X[:, :-1], Y[:, 1:] - Y[:, :-1]
                s = (-ey, ex)
            length = torch.sqrt(ex * ex + ey * ey)
            self.n.append((s[0] / length, s[1] / length))
            self.len.append(length)
        ax_, ay_ = X[1:, 1:] - X[:-1, :-1], Y[1:, 1:] - Y[:-1, :-1]
        bx, by = X[1:, :-1] - X[:-1, 1:], Y[1:, :-1] - Y[:-1, 1:]
        self.area = 0.5 * (ax_ * by - ay_ * bx)


def _residual(f, U):
    nd = f.ndim
    h = [(f.hi[d] - f.lo[d]) / f.n[d] for d in range(nd)]
    R = torch.zeros_like(U)
    m = f.metrics
    for ax in range(nd):
        dim, n = 3 - ax, f.n[ax]
        normals = None
        if m is not None:
            nx, ny = m.n[ax]
            normals = [(nx.select(1 - ax, k).unsqueeze(1 - ax), ny.select(1 - ax, k).unsqueeze(1 - ax)) for k in (0, -1)]
        L, Q = _states(_pad(f, U, ax, 2, normals), dim, n, f.scheme)
        if m is not None:
            nx, ny = m.n[ax]

            def turn(q):
                return torch.stack([q[0], nx * q[1] + ny * q[2], -ny * q[1] + nx * q[2], q[3]])

            G = _roe(turn(L), turn(Q), 0, 2)
            F = torch.stack([G[0], nx * G[1] - ny * G[2], ny * G[1] + nx * G[2], G[3]]) * m.len[ax]
            area = 1.0
        else:
            F = _roe(L, Q, ax, nd)
            area = math.prod(h[d] for d in range(nd) if d != ax)
        if f.mu > 0:
            F = F - _viscous(f, U, ax)
        R = R + (F.narrow(dim, 1, n) - F.narrow(dim, 0, n)) * area
    if f.source is not None:
        R = R - math.prod(h) * f.source
    return R


def _dt(f, U):
    nd = f.ndim
    u = [U[1 + d] / U[0] for d in range(nd)]
    p = (GAMMA - 1) * (U[nd + 1] - 0.5 * U[0] * sum(a * a for a in u))
    c = torch.sqrt(GAMMA * p / U[0])
    if f.metrics is not None:
        m, lam = f.metrics, 0.0
        for ax in (0, 1):
            sx, sy = (m.n[ax][d] * m.len[ax] for d in (0, 1))
            k = f.n[ax]
            sx, sy = (0.5 * (s.narrow(1 - ax, 0, k) + s.narrow(1 - ax, 1, k)) for s in (sx, sy))
            lam = lam + ((u[0] * sx + u[1] * sy).abs() + c * torch.sqrt(sx * sx + sy * sy)) / m.area
    else:
        h = [(f.hi[d] - f.lo[d]) / f.n[d] for d in range(nd)]
        lam = sum((u[d].abs() + c) / h[d] for d in range(nd))
        if f.mu > 0:
            lam = lam + 2 * f.mu / U[0] * max(4 / 3, GAMMA / f.prandtl) * sum(1 / a ** 2 for a in h)
    return f.cfl / lam.max()


def _step(f, U, dt):
    vol = f.metrics.area if f.metrics is not None else math.prod((f.hi[d] - f.lo[d]) / f.n[d] for d in range(f.ndim))
    s = dt / vol
    U1 = U - s * _residual(f, U)
    U2 = 0.75 * U + 0.25 * (U1 - s * _residual(f, U1))
    return U / 3 + 2 / 3 * (U2 - s * _residual(f, U2))


def _exact_flow(case, seed):
    f = Flow(case, seed)
    f.metrics = None if f.nodes is None else _Metrics(f.nodes)
    return f


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step2d", "step3d", "split"):
        f = _exact_flow(case, seed)
        U, dts = f.U, []
        for _ in range(case["steps"]):
            dts.append(_dt(f, U))
            U = _step(f, U, dts[-1])
        out = {"U": U, "dt": torch.stack(dts)}
        if kind == "split":
            out["R"] = _residual(f, U)
        return out
    if kind == "batch":
        parts = []
        for nx, ny, s in _batch_grids(case, seed):
            f = _exact_flow({"kind": "step2d", "flow": "vortex", "nx": nx, "ny": ny, "scheme": case["scheme"]}, s)
            U = f.U
            for _ in range(case["steps"]):
                U = _step(f, U, _dt(f, U))
            parts.append(U.reshape(-1))
        return {"U": torch.cat(parts)}
    if kind == "rollout":
        f = _exact_flow(case, seed)
        U, states, dts = f.U, [], []
        for _ in range(case["steps"]):
            dts.append(_dt(f, U))
            states.append(U)
            U = _step(f, U, dts[-1])
        m = min(case["nx"], case["ny"])
        a, b = m // 2 - m // 16, m // 2 + m // 16
        last = U.clone().requires_grad_(True)
        W = last[:, 0, a:b, a:b]
        p = (GAMMA - 1) * (W[3] - 0.5 * (W[1] ** 2 + W[2] ** 2) / W[0])
        obj = p.sum() * math.prod((f.hi[d] - f.lo[d]) / f.n[d] for d in range(2))
        (lam,) = torch.autograd.grad(obj, last)
        for V, dt in zip(reversed(states), reversed(dts)):
            V = V.clone().requires_grad_(True)
            (lam,) = torch.autograd.grad(_step(f, V, dt), V, lam)
        return {"U": U, "dt": torch.stack(dts), "objective": obj.detach(), "grad": lam}
    P0 = torch.as_tensor(_initial_network(seed, case["n_in"]), device=DEV).float().double()
    if kind == "train":
        return _exact_train(case, seed, P0)
    return _exact_sweep(case, P0)


def _initial_network(seed, n_in):
    """Glorot-uniform weights and biases, layer by layer, from the seed."""
    rng = np.random.default_rng(seed)
    parts = []
    for fi, fo in ((n_in, 64), (64, 64), (64, 64), (64, 1)):
        b = math.sqrt(6.0 / (fi + fo))
        parts += [rng.uniform(-b, b, size=(fo, fi)).ravel(), rng.uniform(-b, b, size=fo)]
    return np.concatenate(parts)


def _layers(P, n_in):
    out, o = [], 0
    for fi, fo in ((n_in, 64), (64, 64), (64, 64), (64, 1)):
        out.append((P[o:o + fi * fo].view(fo, fi), P[o + fi * fo:o + fi * fo + fo]))
        o += fi * fo + fo
    return out


def _forward(P, X, n_in):
    H = X
    ls = _layers(P, n_in)
    for W, b in ls[:-1]:
        H = torch.relu(H @ W.T + b)
    return (H @ ls[-1][0].T + ls[-1][1])[:, 0]


def _exact_train(case, seed, P):
    X, y, order = _train_data(case, seed)
    X, y = (torch.as_tensor(a, device=DEV).double() for a in (X, y))
    hp = {k: float(np.float32(v)) for k, v in dict(lr=9e-4, b1=0.95, b2=0.90, eps=1e-9, alpha=1e-4).items()}
    n, m, v, t, losses = case["rows"], torch.zeros_like(P), torch.zeros_like(P), 0, []
    for e in range(case["epochs"]):
        acc = 0.0
        for s in range(0, n, 200):
            rows = torch.as_tensor(order[e, s:s + 200].astype(np.int64), device=DEV)
            P = P.detach().requires_grad_(True)
            B = len(rows)
            w2 = sum((W * W).sum() for W, _ in _layers(P, case["n_in"]))
            loss = ((_forward(P, X[rows], case["n_in"]) - y[rows]) ** 2).sum() / (2 * B) + hp["alpha"] / (2 * B) * w2
            (g,) = torch.autograd.grad(loss, P)
            acc += float(loss) * B
            t += 1
            m = hp["b1"] * m + (1 - hp["b1"]) * g
            v = hp["b2"] * v + (1 - hp["b2"]) * g * g
            lr = hp["lr"] * math.sqrt(1 - hp["b2"] ** t) / (1 - hp["b1"] ** t)
            P = P.detach() - lr * m / (torch.sqrt(v) + hp["eps"])
        losses.append(acc / n)
    return {"params": P, "m": m, "v": v, "losses": np.array(losses), "pred": _forward(P, X[n:], case["n_in"])}


def _exact_sweep(case, P):
    sp, n_in = _space(case), case["n_in"]
    best = torch.zeros(0, dtype=torch.float64, device=DEV)
    radix = [int(r) for r in sp.radix]
    tab = [torch.tensor([[sp.f1[s][c], sp.f2[s][c]] for c in range(radix[s])], dtype=torch.float64, device=DEV)
           for s in range(len(radix))]
    done = 0
    while done < case["count"]:
        m = min(4_000_000, case["count"] - done)
        rem = torch.arange(m, device=DEV) + (case["begin"] + done)
        cols = []
        for s in range(len(radix)):
            cols.append(tab[s][rem % radix[s]])
            rem = rem // radix[s]
        if n_in == 16:
            cols.append(torch.tensor([sp.extra[0], sp.extra[1]], dtype=torch.float64, device=DEV).expand(m, 2))
        out = _forward(P, torch.cat(cols, 1), n_in)
        best = torch.sort(torch.cat([best, out]))[0][: case["k"]]
        done += m
    return {"index": None, "value": best}
