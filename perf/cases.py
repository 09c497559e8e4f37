"""Performance cases of the library: what its users have it do, through the public
entry points (Solver, Batch, rollout), from a tube of a few hundred cells to
the 4096 x 4096 grid.

listed()             the cases that are timed
draw(rng)            another case of the same ranges
prepare(case, seed)  inputs on the GPU and the handle a program keeps
run(state)           one pass: a call (or the few calls) of a user's program
work(case)           bytes and operations one pass cannot do without
exact(case, seed)    what run returns, from plain torch in 64 bits

The flows are those of the paper's Sec. 3 and of the repository's benchmark:
the Lax tube extruded in y with a density wave on it ("lax"), the
Taylor-Green vortex ("vortex"), smooth periodic random fields ("random") and
a density pulse in gas at rest with open sides ("pulse").  Grid spacings,
time steps and velocity sets are the ones those runs use.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch
import torch.utils.checkpoint

from paper_2502_16818_amd import FP64, MIXED, MIXED_COMP, Batch, Solver
from paper_2502_16818_amd.cdbm import BATCH_ROW_PIECES, make_params
from paper_2502_16818_amd.rollout import rollout

PRECISION = {"fp64": FP64, "mixed": MIXED, "comp": MIXED_COMP}
R2 = math.sqrt(2.0)
# (v_a .. v_d), (eta_a .. eta_d)
SETS = {
    "lax": ((4.4, 4.4, 3.0, 1.8), (0.0, 0.0, 5.0, 0.0)),
    "vortex": ((0.2, 0.2, 2.0, 2.0), (0.0, 5.0, 0.0, 2.6)),
    "random": ((1.4 * R2, 1.1 * R2, 1.1 * R2, 1.0 * R2), (3.0 * R2, 0.0, 0.0, 0.0)),
    "pulse": ((1.4, 1.1, 1.1, 1.0), (3.0, 0.0, 0.0, 0.0)),
}


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # one step of a 32 x 32 grid in a call of its own: the smallest call,
        # all launch latency (coupling codes step once and look at the fields)
        dict(name="call_32", kind="step", flow="random", nx=32, ny=32, precision="mixed", nsteps=1),
        # the 500-cell Riemann tube, a stretch of its thousands of steps
        dict(name="tube_500_fp64", kind="step", flow="lax", nx=500, ny=1, precision="fp64", nsteps=200),
        # a long tube (the Ma = 15 shock tube has 10000 cells) in the throughput form
        dict(name="tube_10000_mixed", kind="step", flow="lax", nx=10000, ny=1, precision="mixed", nsteps=100),
        # the 100 x 100 vortex of Sec. 3.5, in FP64
        dict(name="vortex_100_fp64", kind="step", flow="vortex", nx=100, ny=100, precision="fp64", nsteps=100),
        # the slowly decaying 512 x 512 vortex, which the compensated form is for
        dict(name="vortex_512_comp", kind="step", flow="vortex", nx=512, ny=512, precision="comp", nsteps=40),
        # the 1600 x 1200 sound wave with open sides: four steps between two
        # looks at the field, an ordinary size that is no multiple of a strip
        dict(name="pulse_1600x1200", kind="step", flow="pulse", nx=1600, ny=1200, precision="mixed", nsteps=4),
        # a ragged grid in FP64 (odd width, rows off the cache lines)
        dict(name="lax_2047x1531_fp64", kind="step", flow="lax", nx=2047, ny=1531, precision="fp64", nsteps=4),
        # the throughput workload, 4096 x 4096 in the mixed form
        dict(name="lax_4096_mixed", kind="step", flow="lax", nx=4096, ny=4096, precision="mixed", nsteps=8),
        # the ensemble of 96 periodic grids of 128^2 .. 1024^2, in the row-piece
        # layout that tuning picks for it
        dict(name="ensemble_96", kind="batch", grids=96, nmin=128, nmax=1024, precision="mixed", rows=320, tail=96, nsteps=6),
        # the gradient workload: rollout forward and backward on 256 x 256
        dict(name="gradient_256", kind="gradient", n=256, precision="mixed", nsteps=40, every=20),
        # the transpose of one FP64 step on an uneven mid-size grid
        dict(name="adjoint_1000x777", kind="adjoint", flow="random", nx=1000, ny=777, precision="fp64"),
        # diagnostics of a state: fields, nonequilibrium measures, totals
        dict(name="diagnostics_2048", kind="diagnostics", flow="random", nx=2048, ny=2048, precision="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["tube", "small", "mid", "mid", "large", "large", "batch", "gradient", "adjoint", "diagnostics"])
    if kind == "tube":
        return dict(kind="step", flow="lax", nx=_log_int(rng, 200, 10000), ny=1, precision=rng.choice(["fp64", "mixed", "comp"]), nsteps=rng.randint(40, 200))
    if kind == "small":
        return dict(kind="step", flow=rng.choice(["vortex", "random", "pulse"]), nx=_log_int(rng, 20, 200), ny=_log_int(rng, 20, 200), precision=rng.choice(["fp64", "mixed", "comp"]), nsteps=rng.choice([1, rng.randint(2, 100)]))
    if kind == "mid":
        return dict(kind="step", flow=rng.choice(["lax", "vortex", "random", "pulse"]), nx=_log_int(rng, 200, 1600), ny=_log_int(rng, 200, 1600), precision=rng.choice(["fp64", "mixed", "comp"]), nsteps=rng.randint(1, 40))
    if kind == "large":
        return dict(kind="step", flow=rng.choice(["lax", "random", "pulse"]), nx=_log_int(rng, 1200, 4000), ny=_log_int(rng, 1200, 4000), precision=rng.choice(["fp64", "mixed"]), nsteps=rng.randint(1, 4))
    if kind == "batch":
        rows, tail = rng.choice([(0, 0), (192, 64), (320, 96), (448, 160)])
        return dict(kind="batch", grids=_log_int(rng, 4, 90), nmin=rng.choice([64, 100, 128]), nmax=rng.choice([512, 900, 1024]), precision=rng.choice(["fp64", "mixed"]), rows=rows, tail=tail, nsteps=rng.randint(1, 3))
    if kind == "gradient":
        n = _log_int(rng, 48, 400)
        return dict(kind="gradient", n=n, precision=rng.choice(["fp64", "mixed"]), nsteps=rng.randint(8, 30), every=rng.randint(4, 15))
    if kind == "adjoint":
        return dict(kind="adjoint", flow=rng.choice(["lax", "random", "pulse"]), nx=_log_int(rng, 64, 1800), ny=_log_int(rng, 64, 1800), precision=rng.choice(["fp64", "mixed"]))
    return dict(kind="diagnostics", flow=rng.choice(["lax", "vortex", "random"]), nx=_log_int(rng, 64, 3000), ny=_log_int(rng, 64, 3000), precision=rng.choice(["fp64", "mixed", "comp"]))


# ---------------------------------------------------------------- inputs

def _device():
    return torch.device("cuda", torch.cuda.current_device())


def _centres(n):
    return (torch.arange(n, dtype=torch.float64, device=_device()) + 0.5) / n


def _waves(rng, nx, ny, modes=5):
    """Periodic sum of plane waves on the unit square, largest value 1."""
    X, Y = _centres(nx)[None, :], _centres(ny)[:, None]
    s = torch.zeros((ny, nx), dtype=torch.float64, device=_device())
    for _ in range(modes):
        kx, ky = rng.integers(1, 5, size=2)
        s += rng.uniform(0.2, 1.0) * torch.cos(2 * math.pi * (int(kx) * X + int(ky) * Y) + rng.uniform(0.0, 2 * math.pi))
    return s / s.abs().max()


def _flow(flow, nx, ny, seed):
    """(parameters without nx, ny, precision; fields rho, u_x, u_y, T) of a flow."""
    rng = np.random.default_rng(seed)
    v, eta = SETS[flow]
    full = lambda c: torch.full((ny, nx), float(c), dtype=torch.float64, device=_device())
    if flow == "lax":
        left = (_centres(nx) < 0.5)[None, :].expand(ny, nx)
        w = _centres(nx)[None, :] * 2 + _centres(ny)[:, None] * (3 if ny > 1 else 0)
        rho = torch.where(left, full(0.445), full(0.5)) * (1 + 1e-3 * torch.cos(2 * math.pi * w + rng.uniform(0, 2 * math.pi)))
        fields = (rho, torch.where(left, full(0.698), full(0.0)), full(0.0), torch.where(left, full(7.928), full(1.142)))
        par = dict(dx=2e-3, dy=2e-3, dt=2e-5, tau=1e-4, gamma=float(rng.choice([1.4, 5.0 / 3.0])), bc_x=1, bc_y=0)
    elif flow == "vortex":
        X, Y = 2 * math.pi * _centres(nx)[None, :] + rng.uniform(0, 6), 2 * math.pi * _centres(ny)[:, None] + rng.uniform(0, 6)
        p = 1 + 0.0025 * (torch.cos(2 * X) + torch.cos(2 * Y))
        fields = (full(1.0), 0.1 * torch.sin(X) * torch.cos(Y), -0.1 * torch.cos(X) * torch.sin(Y), p)
        d = 2 * math.pi / max(nx, ny)
        par = dict(dx=d, dy=d, dt=1e-4, tau=1e-4, gamma=1.4, bc_x=0, bc_y=0)
    elif flow == "random":
        u, w = _waves(rng, nx, ny), _waves(rng, nx, ny)
        scale = 0.29 / torch.sqrt(u * u + w * w).max()
        fields = (1.25 + 0.75 * _waves(rng, nx, ny), u * scale, w * scale, 1.25 + 0.75 * _waves(rng, nx, ny))
        par = dict(dx=1.0 / max(nx, 256), dy=1.0 / max(ny, 256), dt=1e-5, tau=float(10 ** rng.uniform(-4.5, -3.0)), gamma=float(rng.uniform(1.1, 1.67)), bc_x=0, bc_y=0)
    else:
        x0, y0 = rng.uniform(0.3, 0.7), rng.uniform(0.3, 0.7)
        r2 = ((_centres(nx)[None, :] - x0) * nx) ** 2 + ((_centres(ny)[:, None] - y0) * ny) ** 2
        fields = (1 + 0.1 * torch.exp(-r2 / (2 * (0.1 * max(nx, ny)) ** 2)), full(0.0), full(0.0), full(1.0))
        par = dict(dx=5e-4, dy=5e-4, dt=2e-5, tau=1e-4, gamma=1.4, bc_x=1, bc_y=1)
    return dict(par, v=v, eta=eta), tuple(t.contiguous() for t in fields)


def _params(par, nx, ny, precision):
    return make_params(nx=nx, ny=ny, precision=PRECISION[precision], **par)


def _off_equilibrium(nx, ny, seed):
    """A smooth factor per velocity, within 2 % of 1: a state away from equilibrium."""
    rng = np.random.default_rng(seed + 77)
    return torch.stack([1 + 0.02 * _waves(rng, nx, ny, modes=2) for _ in range(16)])


def _sizes(case):
    step = 64 if case["nmin"] % 64 == 0 else 20
    k = np.random.default_rng(case["grids"]).integers(0, (case["nmax"] - case["nmin"]) // step + 1, size=case["grids"])
    return [int(i) * step + case["nmin"] for i in k]


def _grids(case, seed):
    """The batch's grids: sizes that belong to the case, flows to the seed."""
    rng = np.random.default_rng(seed)
    out = []
    for n in _sizes(case):
        par, fields = _flow("random", n, n, int(rng.integers(1 << 30)))
        par.update(dx=1.0 / n, dy=1.0 / n, tau=float(10.0 ** rng.uniform(-4.5, -3)))
        out.append((par, n, fields))
    return out


def _adjoint_vector(nx, ny, seed):
    g = torch.Generator(device=_device()).manual_seed(seed + 5)
    return torch.randn((16, ny, nx), dtype=torch.float64, device=_device(), generator=g)


def _gradient(case, seed):
    n = case["n"]
    par, fields = _flow("random", n, n, seed)
    par.update(dx=1.0 / n, dy=1.0 / n, dt=2e-5 if n <= 256 else 1e-5, tau=1e-4, gamma=1.4)
    rng = np.random.default_rng(seed + 1)
    return par, fields, fields[0] * (1 + 0.01 * _waves(rng, n, n))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        par, fields = _flow(case["flow"], case["nx"], case["ny"], seed)
        s = Solver(_params(par, case["nx"], case["ny"], case["precision"]))
        return dict(kind=kind, s=s, f=s.init(*fields), out=s.empty_f(), nsteps=case["nsteps"])
    if kind == "batch":
        grids = _grids(case, seed)
        b = Batch([_params(par, n, n, case["precision"]) for par, n, _ in grids])
        if case["rows"]:
            b.set_launch(BATCH_ROW_PIECES, 0, case["rows"], case["tail"])
        return dict(kind=kind, s=b, f=b.init([fl for _, _, fl in grids]), out=b.empty_f(), nsteps=case["nsteps"])
    if kind == "gradient":
        par, fields, target = _gradient(case, seed)
        s = Solver(_params(par, case["n"], case["n"], case["precision"]))
        tau = torch.tensor(par["tau"], dtype=torch.float64, device=_device())
        leaves = [t.clone().requires_grad_(True) for t in (*fields, tau)]
        return dict(kind=kind, s=s, leaves=leaves, target=target, nsteps=case["nsteps"], every=case["every"])
    par, fields = _flow(case["flow"], case["nx"], case["ny"], seed)
    s = Solver(_params(par, case["nx"], case["ny"], case["precision"]))
    f = s.init(*fields)
    f[:16].mul_(_off_equilibrium(case["nx"], case["ny"], seed).to(f.dtype))
    if kind == "adjoint":
        return dict(kind=kind, s=s, f=f, lam=_adjoint_vector(case["nx"], case["ny"], seed), out=s.empty_lam())
    return dict(kind=kind, s=s, f=f)


# ---------------------------------------------------------------- one pass

def run(state):
    s, kind = state["s"], state["kind"]
    if kind in ("step", "batch"):
        return s.step(state["f"], state["out"], nsteps=state["nsteps"])
    if kind == "gradient":
        rho, ux, uy, T = rollout(s, *state["leaves"], state["nsteps"], state["every"])
        loss = ((rho - state["target"]) ** 2).mean()
        grads = torch.autograd.grad(loss, state["leaves"])
        return dict(fields=[rho.detach(), ux.detach(), uy.detach(), T.detach()], loss=loss.detach(), grads=list(grads))
    if kind == "adjoint":
        lam, dtau = s.step_adjoint(state["f"], state["lam"], state["out"])
        return dict(lam=lam, dtau=dtau)
    f = state["f"]
    return dict(fields=list(s.moments(f)), tne=s.tne(f), totals=s.totals(f))


# ---------------------------------------------------------------- work

# additions and multiplications of one cell and Runge-Kutta stage: moments 80,
# equilibrium and relaxation 250, flux differences 24 x 9, combination 32
STAGE_FLOPS = 580


def _state_bytes(precision):
    return {"fp64": 128, "mixed": 64, "comp": 80}[precision]


def work(case):
    kind = case["kind"]
    if kind == "step":
        # every step reads the state and writes the next one
        n = case["nx"] * case["ny"] * case["nsteps"]
        return {"bytes": 2 * _state_bytes(case["precision"]) * n, "flops": 2 * STAGE_FLOPS * n}
    if kind == "batch":
        n = sum(m * m for m in _sizes(case)) * case["nsteps"]
        return {"bytes": 2 * _state_bytes(case["precision"]) * n, "flops": 2 * STAGE_FLOPS * n}
    if kind == "gradient":
        # per step: the state in and out twice (forward, and its recomputation
        # from a checkpoint), the state and the FP64 adjoint in, the adjoint out
        n = case["n"] ** 2 * case["nsteps"]
        return {"bytes": (5 * _state_bytes(case["precision"]) + 2 * 128) * n, "flops": 9 * STAGE_FLOPS * n}
    n = case["nx"] * case["ny"]
    if kind == "adjoint":
        return {"bytes": (_state_bytes(case["precision"]) + 2 * 128) * n, "flops": 5 * STAGE_FLOPS * n}
    return {"bytes": (3 * _state_bytes(case["precision"]) + 8 * (4 + 12)) * n, "flops": 900 * n}


# ---------------------------------------------------------------- 64-bit reference

class _Ref:
    """The method in plain torch, float64: raw Maxwellian moments through the
    inverse of the 16 x 16 moment matrix, NND differences by rolled copies."""

    SX = (1, 0, -1, 0, 1, -1, -1, 1) * 2
    SY = (0, 1, 0, -1, 1, 1, -1, -1) * 2

    def __init__(self, par, nx, ny):
        self.par, self.nx, self.ny = par, nx, ny
        self.vx = [par["v"][i // 4] * self.SX[i] for i in range(16)]
        self.vy = [par["v"][i // 4] * self.SY[i] for i in range(16)]
        self.e2 = [par["eta"][i // 4] ** 2 for i in range(16)]
        M = np.array([self._psi(self.vx[i], self.vy[i], self.vx[i] ** 2 + self.vy[i] ** 2 + self.e2[i]) for i in range(16)], dtype=np.float64).T
        inv = np.linalg.inv(M)
        inv = inv @ (2 * np.eye(16) - M @ inv)
        self.inv = torch.tensor(inv, device=_device())
        self.a = 2.0 / (par["gamma"] - 1.0)   # D + I

    @staticmethod
    def _psi(x, y, e):
        one = x * 0 + 1.0
        return [one, x, y, e * one, x * x, x * y, y * y, e * x, e * y, x * x * x, x * x * y, x * y * y, y * y * y, e * x * x, e * x * y, e * y * y]

    def macro(self, f, r=None):
        q = [sum(f[i] * w[i] for i in range(16)) for w in ([1.0] * 16, self.vx, self.vy, [self.vx[i] ** 2 + self.vy[i] ** 2 + self.e2[i] for i in range(16)])]
        if r is not None:
            q = [a + b for a, b in zip(q, r)]
        ux, uy = q[1] / q[0], q[2] / q[0]
        return q[0], ux, uy, (q[3] / q[0] - ux * ux - uy * uy) / self.a

    def feq(self, rho, ux, uy, T):
        a = self.a
        A2, A4 = ux * ux + uy * uy + (a + 2) * T, ux * ux + uy * uy + (a + 4) * T
        m = [torch.ones_like(ux), ux, uy, ux * ux + uy * uy + a * T, ux * ux + T, ux * uy, uy * uy + T, ux * A2, uy * A2,
             ux * (ux * ux + 3 * T), uy * (ux * ux + T), ux * (uy * uy + T), uy * (uy * uy + 3 * T),
             ux * ux * A4 + T * A2, ux * uy * A4, uy * uy * A4 + T * A2]
        m = torch.stack([rho * t for t in m]).reshape(16, -1)
        return (self.inv @ m).reshape(16, self.ny, self.nx)

    def _sh(self, t, o, dim, bc):
        """Value at the cell `o` further along, through the boundary condition."""
        n = t.shape[dim]
        at = torch.arange(n, device=t.device) + o
        at = at % n if bc == 0 else at.clamp(0, n - 1)
        return t.index_select(dim, at)

    @staticmethod
    def _mm(X, Y):
        same = ((X > 0) & (Y > 0)) | ((X < 0) & (Y < 0))
        return torch.where(same, torch.where(X.abs() <= Y.abs(), X, Y), torch.zeros_like(X))

    def _nnd(self, t, s, dim, bc):
        at = lambda o: t if o == 0 else self._sh(t, o, dim, bc)
        if s > 0:
            d0 = t - at(-1)
            return d0 + 0.5 * (self._mm(at(1) - t, d0) - self._mm(d0, at(-1) - at(-2)))
        d1 = at(1) - t
        return d1 - 0.5 * (self._mm(at(2) - at(1), d1) - self._mm(d1, t - at(-1)))

    def stage(self, f, tau):
        """f + dt L(f)"""
        p = self.par
        eq = self.feq(*self.macro(f))
        out = []
        for i in range(16):
            d = -(p["dt"] / tau) * (f[i] - eq[i])
            if self.SX[i]:
                d = d - p["dt"] * self.vx[i] / p["dx"] * self._nnd(f[i], self.SX[i], 1, p["bc_x"])
            if self.SY[i]:
                d = d - p["dt"] * self.vy[i] / p["dy"] * self._nnd(f[i], self.SY[i], 0, p["bc_y"])
            out.append(f[i] + d)
        return torch.stack(out)

    def step(self, f, tau=None):
        tau = self.par["tau"] if tau is None else tau
        return 0.5 * f + 0.5 * self.stage(self.stage(f, tau), tau)

    def tne(self, f, r=None):
        rho, ux, uy, T = self.macro(f, r)
        d = f - self.feq(rho, ux, uy, T)
        out = [0.0] * 12
        for i in range(16):
            x, y = self.vx[i] - ux, self.vy[i] - uy
            psi = self._psi(x, y, x * x + y * y + self.e2[i])[4:]
            out = [o + d[i] * w for o, w in zip(out, psi)]
        return torch.stack(out)


def _stored(f, precision):
    return f if precision == "fp64" else f.float().double()


def _exact_steps(par, nx, ny, fields, precision, nsteps):
    ref = _Ref(par, nx, ny)
    f0 = ref.feq(*fields)
    f = _stored(f0, precision) if precision == "mixed" else f0
    for _ in range(nsteps):
        f = ref.step(f)
    # a compensated state is f rounded to float and four planes of the
    # conserved moments that rounding removed, which in exact arithmetic are 0
    return torch.cat([f, torch.zeros_like(f[:4])]) if precision == "comp" else f


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        if case["nsteps"] * (0.02 + case["nx"] * case["ny"] * 1.5e-8) > 18:
            return None
        par, fields = _flow(case["flow"], case["nx"], case["ny"], seed)
        return _exact_steps(par, case["nx"], case["ny"], fields, case["precision"], case["nsteps"])
    if kind == "batch":
        return torch.cat([_exact_steps(par, n, n, fl, case["precision"], case["nsteps"]).reshape(-1) for par, n, fl in _grids(case, seed)])
    if kind == "gradient":
        n = case["n"]
        par, fields, target = _gradient(case, seed)
        ref = _Ref(par, n, n)
        leaves = [t.clone().requires_grad_(True) for t in (*fields, torch.tensor(par["tau"], dtype=torch.float64, device=_device()))]
        f = ref.feq(*leaves[:4])
        for _ in range(case["nsteps"]):
            f = torch.utils.checkpoint.checkpoint(ref.step, f, leaves[4], use_reentrant=False)
        out = ref.macro(f)
        loss = ((out[0] - target) ** 2).mean()
        grads = torch.autograd.grad(loss, leaves)
        return dict(fields=[t.detach() for t in out], loss=loss.detach(), grads=list(grads))
    nx, ny = case["nx"], case["ny"]
    par, fields = _flow(case["flow"], nx, ny, seed)
    ref = _Ref(par, nx, ny)
    f0 = ref.feq(*fields)
    f = _stored(f0, case["precision"])
    w = _off_equilibrium(nx, ny, seed)
    f = f * w if case["precision"] == "fp64" else (f.float() * w.float()).double()
    if kind == "adjoint":
        f = f.requires_grad_(True)
        tau = torch.tensor(par["tau"], dtype=torch.float64, device=_device(), requires_grad=True)
        g = torch.autograd.grad(ref.step(f, tau), (f, tau), _adjoint_vector(nx, ny, seed))
        return dict(lam=g[0], dtau=g[1].reshape(1))
    r = None
    if case["precision"] == "comp":   # the conserved moments that rounding the initial f removed
        d = f0 - f0.float().double()
        r = [sum(d[i] * k[i] for i in range(16)) for k in ([1.0] * 16, ref.vx, ref.vy, [ref.vx[i] ** 2 + ref.vy[i] ** 2 + ref.e2[i] for i in range(16)])]
    q = ref.macro(f, r)
    totals = torch.stack([t.sum() for t in (q[0], q[0] * q[1], q[0] * q[2], q[0] * (ref.a * q[3] + q[1] ** 2 + q[2] ** 2))])
    return dict(fields=list(q), tne=ref.tne(f, r), totals=totals)
