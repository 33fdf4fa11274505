"""The calls whose time matters to a program that uses this library.

A case names an operation, a grid and the options of its plan:

  poisson   one pressure-Poisson solve (`Plan.poisson_solve`)
  step      one projection step (`Plan.projection_step`)
  loop      a time loop of several steps (`Plan.run_steps`), restarted from a
            stored field, with plane statistics and with or without graphs
  grad      one differentiable step forward and backward
            (`autograd.projection_step`)
  rollout   several differentiable steps with checkpoints, forward and backward
            (`autograd.rollout`)

Grids run from 64^3 (launch latency) through ragged ones (lengths 3 * 2^a, row
counts that no partition count divides) to the largest Poisson workload of the
bench.  Inputs are the perturbed laminar channel flow of the step workloads and
the divergent k^-5/3 field of the large Poisson workload, made on the device.
"""
import functools
import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_2104_08863_amd import autograd, synth
from paper_2104_08863_amd.api import Plan

F64 = torch.float64
NU = 1.0 / 550.0
FX = 3.0 / 550.0


def _case(name, op, nx, ny, nz, precision="fp64", gamma=2.5, solver="pdd", field="uniform", steps=1, every=1,
          pressure=False, graph=False, stats=0):
    return {"name": name, "op": op, "nx": nx, "ny": ny, "nz": nz, "precision": precision, "gamma": gamma,
            "solver": solver, "field": field, "steps": steps, "every": every, "pressure": pressure, "graph": graph,
            "stats": stats}


def listed():
    return [
        # the smallest grid in use: one solve of a coarse box, bound by launches
        _case("poisson_fp64_64", "poisson", 64, 64, 64, gamma=2.0),
        # an ordinary grid whose lengths are 3 * 2^a and whose 130 rows no partition count divides
        _case("poisson_fp64_ragged", "poisson", 192, 130, 96),
        # the pressure solve of the Re_tau = 550 shaped channel
        _case("poisson_fp64_large", "poisson", 1024, 256, 512),
        # uniform wall-normal spacing (a box without clustering), transform solve in y
        _case("poisson_fp64_uniform_y", "poisson", 512, 256, 256, gamma=0.0, solver="dct"),
        # the Re_tau = 1000 shaped solve in mixed precision with one refinement: the largest call
        _case("poisson_mixed_largest", "poisson", 2048, 512, 1536, precision="mixed", gamma=2.6, field="powerlaw"),
        # the step of the Re_tau = 550 shaped channel
        _case("step_fp64_large", "step", 1024, 256, 512),
        # a step on a ragged grid that also returns the pressure
        _case("step_fp64_ragged", "step", 384, 97, 192, pressure=True),
        # a single-precision state with the mixed pressure solve
        _case("step_mixed", "step", 512, 192, 512, precision="mixed", gamma=3.0),
        # a short averaging window on a coarse grid, replayed from graphs
        _case("loop_fp64_64_graph", "loop", 64, 64, 64, gamma=2.0, steps=20, graph=True, stats=5),
        # sensitivities: one step and its adjoint on the large grid, in both precisions
        _case("grad_fp64_large", "grad", 1024, 256, 512),
        _case("grad_mixed_large", "grad", 1024, 384, 1024, precision="mixed", gamma=3.0),
        # an optimisation through eight checkpointed steps
        _case("rollout_fp64_256", "rollout", 256, 128, 256, gamma=2.0, steps=8, every=2),
    ]


_LENGTHS = [32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024]
# most points of a drawn grid, by operation
_MOST = {"poisson": 1 << 27, "step": 1 << 26, "loop": 1 << 22, "grad": 1 << 25, "rollout": 1 << 22}


def draw(rng):
    op = rng.choice(["poisson", "poisson", "step", "step", "loop", "grad", "rollout"])
    c = _case("", op, 0, 0, 0, gamma=round(rng.uniform(1.5, 3.0), 3))
    del c["name"]
    points = math.exp(rng.uniform(math.log(1 << 17), math.log(_MOST[op])))
    while True:
        nx, nz = rng.choice(_LENGTHS), rng.choice(_LENGTHS)
        ny = int(round(points / (nx * nz)))
        if 24 <= ny <= 512 and nx * ny * nz <= _MOST[op]:
            break
    c.update(nx=nx, ny=ny, nz=nz)
    if op != "loop" and rng.random() < 0.35:
        c["precision"] = "mixed"
    if op == "poisson":
        c["field"] = rng.choice(["uniform", "powerlaw"])
        if c["precision"] == "fp64" and rng.random() < 0.2:
            c.update(gamma=0.0, solver="dct", ny=min((n for n in _LENGTHS if n <= 512), key=lambda n: abs(n - ny)))
            if nx * c["ny"] * nz > _MOST[op]:
                c["ny"] = 64
    elif op == "step":
        c["pressure"] = c["precision"] == "fp64" and rng.random() < 0.3
    elif op == "loop":
        c.update(steps=rng.randint(2, 12), graph=rng.random() < 0.5, stats=rng.choice([0, 1, 4]))
    elif op == "rollout":
        c.update(steps=rng.randint(2, 4), every=rng.randint(1, 3))
    return c


# ------------------------------------------------------------------ inputs
def _points(c):
    return c["nx"] * c["ny"] * c["nz"]


def _box(c):
    """Lengths (4 pi x 2 pi where the grid is that fine, else 2 pi x pi) and wall-normal faces."""
    big = c["nx"] >= 1024
    return (4 * math.pi, 2 * math.pi) if big else (2 * math.pi, math.pi), synth.tanh_faces(c["ny"], c["gamma"])


def _dt(c):
    """A stable time step of the perturbed laminar flow (advective and viscous limits of the explicit scheme)."""
    (lx, lz), yf = _box(c)
    dx, dz, dy = lx / c["nx"], lz / c["nz"], float(np.diff(yf).min())
    return 0.2 / (2.0 / dx + 0.5 / dy + 0.5 / dz + 4.0 * NU * (1 / dx**2 + 1 / dy**2 + 1 / dz**2))


def _poiseuille(c, gen):
    """U = 1.5 (1 - y^2) plus N(0, 0.1^2) on every velocity unknown; the top-wall v plane is 0."""
    dtype = F64 if c["precision"] == "fp64" else torch.float32
    shape = (c["ny"], c["nz"], c["nx"])
    _, yf = _box(c)
    yc = torch.tensor(0.5 * (yf[1:] + yf[:-1]), dtype=dtype, device="cuda")
    u, v, w = (torch.randn(shape, dtype=dtype, device="cuda", generator=gen).mul_(0.1) for _ in range(3))
    u += (1.5 * (1 - yc * yc))[:, None, None]
    v[-1] = 0
    return u, v, w


def _source(c, gen):
    """A right-hand side of the Poisson equation: U[-1, 1], or the divergence-shaped field whose horizontal
    amplitude follows k^(1 - 4/3), with random phases and white in y."""
    shape = (c["ny"], c["nz"], c["nx"])
    f = torch.rand(shape, dtype=F64, device="cuda", generator=gen).mul_(2).sub_(1)
    if c["field"] == "powerlaw":
        kx = torch.arange(c["nx"] // 2 + 1, dtype=F64, device="cuda")
        kz = torch.fft.fftfreq(c["nz"], d=1.0 / c["nz"], dtype=F64, device="cuda")
        k = torch.sqrt(kx[None, :] ** 2 + kz[:, None] ** 2)
        amp = k * torch.clamp(k, min=1.0) ** (-4.0 / 3.0)
        amp *= math.sqrt(c["nx"] * c["nz"]) / float(torch.linalg.norm(amp))
        for j0 in range(0, c["ny"], 32):
            f[j0:j0 + 32] = torch.fft.irfft2(torch.fft.rfft2(f[j0:j0 + 32]).mul_(amp), s=shape[1:])
    return f


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return (_source(c, gen),) if c["op"] == "poisson" else _poiseuille(c, gen)


def _cotangent(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 1_000_003)
    dtype = F64 if c["precision"] == "fp64" else torch.float32
    shape = (c["ny"], c["nz"], c["nx"])
    g = tuple(torch.randn(shape, dtype=dtype, device="cuda", generator=gen) for _ in range(3))
    g[1][-1] = 0
    return g


def prepare(case, seed):
    c = case
    (lx, lz), yf = _box(c)
    op = c["op"]
    plan = Plan(c["nx"], c["ny"], c["nz"], lx, lz, yf, precision=c["precision"], y_solver=c["solver"],
                step=op in ("step", "loop"), adjoint=op in ("grad", "rollout"))
    x = _inputs(c, seed)
    s = {"case": c, "plan": plan, "x": x, "dt": _dt(c)}
    if op == "poisson":
        s["out"] = torch.empty_like(x[0])
    elif op == "step":
        s["out"] = tuple(torch.empty_like(t) for t in x)
        s["p"] = torch.empty(x[0].shape, dtype=F64, device="cuda") if c["pressure"] else None
    elif op == "loop":
        s["state"] = tuple(torch.empty_like(t) for t in x)
        s["work"] = tuple(torch.empty_like(t) for t in x)
        s["stats"] = torch.zeros(c["ny"], 6, dtype=F64, device="cuda")
    else:
        s["g"] = _cotangent(c, seed)
        for t in x:
            t.requires_grad_(True)
    return s


def run(state):
    s, c, plan = state, state["case"], state["plan"]
    op = c["op"]
    if op == "poisson":
        return plan.poisson_solve(s["x"][0], out=s["out"])
    if op == "step":
        out = plan.projection_step(*s["x"], s["dt"], NU, FX, out=s["out"], p=s["p"])
        return out if s["p"] is None else (*out, s["p"])
    if op == "loop":
        for a, b in zip(s["state"], s["x"]):
            a.copy_(b)
        s["stats"].zero_()
        out = plan.run_steps(*s["state"], c["steps"], s["dt"], NU, FX, work=s["work"], stats_every=c["stats"],
                             stats=s["stats"] if c["stats"] else None, use_graph=c["graph"])
        return (*out, s["stats"])
    if op == "grad":
        out = autograd.projection_step(plan, *s["x"], s["dt"], NU, FX)
    else:
        out = autograd.rollout(plan, *s["x"], c["steps"], s["dt"], NU, FX, checkpoint_every=c["every"])
    grads = torch.autograd.grad(out, s["x"], s["g"])
    return (*(t.detach() for t in out), *grads)


def work(case):
    c = case
    n = _points(c)
    es = 8 if c["precision"] == "fp64" else 4
    solve = 5.0 * (math.log2(c["nx"]) + math.log2(c["nz"])) + 16.0
    step = solve + 2 * 110.0 + 12.0
    adjoint = solve + 110.0 + 2 * 160.0 + 12.0
    if c["op"] == "poisson":
        return {"bytes": 16.0 * n, "flops": solve * n}
    if c["op"] == "step":
        return {"bytes": (6.0 * es + (8.0 if c["pressure"] else 0.0)) * n, "flops": step * n}
    if c["op"] == "loop":
        return {"bytes": 6.0 * es * n * c["steps"], "flops": step * n * c["steps"]}
    # forward steps (and those recomputed from checkpoints) read and write the state; an adjoint step reads the
    # state and the gradient and writes the gradient
    again = c["steps"] - -(-c["steps"] // c["every"]) if c["op"] == "rollout" else 0
    return {"bytes": (6.0 * es * (c["steps"] + again) + 9.0 * es * c["steps"]) * n,
            "flops": (step * (c["steps"] + again) + adjoint * c["steps"]) * n}


# ------------------------------------------------------------------ the same in plain torch, 64 bits
class _Box:
    def __init__(self, c):
        (lx, lz), yf = _box(c)
        self.nx, self.ny, self.nz = c["nx"], c["ny"], c["nz"]
        self.dx, self.dz = lx / c["nx"], lz / c["nz"]
        yc = 0.5 * (yf[1:] + yf[:-1])
        dy, dyc = np.diff(yf), np.diff(yc)
        a, b = np.zeros(self.ny), np.zeros(self.ny)
        a[1:], b[:-1] = 1 / (dy[1:] * dyc), 1 / (dy[:-1] * dyc)
        self.lower, self.upper = a, b
        on = functools.partial(torch.tensor, dtype=F64, device="cuda")
        self.dy, self.dyc = on(dy)[:, None, None], on(dyc)[:, None, None]
        self.wl, self.wu = on(dy[1:] / (dy[1:] + dy[:-1]))[:, None, None], on(dy[:-1] / (dy[1:] + dy[:-1]))[:, None, None]
        kx, kz = np.arange(self.nx // 2 + 1), np.arange(self.nz)
        self.k2 = on((2 * np.sin(np.pi * kz / self.nz) / self.dz)[:, None] ** 2
                     + (2 * np.sin(np.pi * kx / self.nx) / self.dx)[None, :] ** 2)


def _solve_lines(b, fh):
    """Thomas along dim 0 of every (kz, kx) line, in place; the singular line with zero weighted mean."""
    ny, a, c = b.ny, b.lower, b.upper
    dy = b.dy[:, 0, 0]
    mean = fh[:, 0, 0] - (dy * fh[:, 0, 0]).sum() / dy.sum()
    k2 = b.k2.clone()
    k2[0, 0] = 1.0
    cp = torch.empty(fh.shape, dtype=F64, device=fh.device)
    for j in range(ny):
        den = -(a[j] + c[j]) - k2
        if j:
            den = den - a[j] * cp[j - 1]
            fh[j] -= a[j] * fh[j - 1]
        torch.div(torch.full_like(den, c[j]), den, out=cp[j])
        fh[j] /= den
    for j in range(ny - 2, -1, -1):
        fh[j] -= cp[j] * fh[j + 1]
    # two sums: the flux at the face above row j, then the differences of p
    flux = torch.cumsum(dy * mean, 0)[:-1] * b.dyc[:, 0, 0]
    line = torch.cat([torch.zeros_like(flux[:1]), torch.cumsum(flux, 0)])
    fh[:, 0, 0] = line - (dy * line).sum() / dy.sum()
    return fh


def _poisson64(b, f):
    fh = torch.fft.fft(torch.fft.rfft(f, dim=2), dim=1)
    return torch.fft.irfft(torch.fft.ifft(_solve_lines(b, fh), dim=1), n=b.nx, dim=2)


class _Solve(torch.autograd.Function):
    """The solve with its transpose: it is self-adjoint under the cell heights."""

    @staticmethod
    def forward(ctx, b, f):
        ctx.b = b
        return _poisson64(b, f)

    @staticmethod
    def backward(ctx, g):
        return None, _poisson64(ctx.b, g / ctx.b.dy) * ctx.b.dy


def _wall(v):
    return torch.cat([v[:-1], torch.zeros_like(v[:1])])


def _below(q):
    return torch.cat([torch.zeros_like(q[:1]), q[:-1]])


def _divergence64(b, u, v, w):
    v = _wall(v)
    return (u - u.roll(1, 2)) / b.dx + (v - _below(v)) / b.dy + (w - w.roll(1, 1)) / b.dz


def _rhs64(b, u, v, w):
    v = _wall(v)
    zero = torch.zeros_like(u[:1])
    uc, wc, vc = 0.5 * (u + u.roll(1, 2)), 0.5 * (w + w.roll(1, 1)), 0.5 * (v + _below(v))
    exy = torch.cat([(u[:-1] * b.wl + u[1:] * b.wu) * 0.5 * (v[:-1] + v[:-1].roll(-1, 2)), zero])
    eyz = torch.cat([(w[:-1] * b.wl + w[1:] * b.wu) * 0.5 * (v[:-1] + v[:-1].roll(-1, 1)), zero])
    exz = 0.25 * (u + u.roll(-1, 1)) * (w + w.roll(-1, 2))

    def flat(q):
        return (q.roll(-1, 2) - 2 * q + q.roll(1, 2)) / b.dx**2 + (q.roll(-1, 1) - 2 * q + q.roll(1, 1)) / b.dz**2

    def centre(q):
        flux = torch.cat([2 * q[:1] / b.dy[0], (q[1:] - q[:-1]) / b.dyc, -2 * q[-1:] / b.dy[-1]])
        return (flux[1:] - flux[:-1]) / b.dy

    ru = -(((uc * uc).roll(-1, 2) - uc * uc) / b.dx + (exy - _below(exy)) / b.dy + (exz - exz.roll(1, 1)) / b.dz)
    ru = ru + NU * (flat(u) + centre(u)) + FX
    rw = -((exz - exz.roll(1, 2)) / b.dx + (eyz - _below(eyz)) / b.dy + ((wc * wc).roll(-1, 1) - wc * wc) / b.dz)
    rw = rw + NU * (flat(w) + centre(w))
    vv, fl = vc * vc, (v - _below(v)) / b.dy
    rv = -((exy - exy.roll(1, 2)) / b.dx + (eyz - eyz.roll(1, 1)) / b.dz)[:-1]
    rv = rv - (vv[1:] - vv[:-1]) / b.dyc + NU * (flat(v)[:-1] + (fl[1:] - fl[:-1]) / b.dyc)
    return ru, torch.cat([rv, zero]), rw


def _step64(b, dt, u, v, w):
    """(u1, v1, w1, p) of one step."""
    v = _wall(v)
    lean = functools.partial(checkpoint, _rhs64, b, use_reentrant=False) if u.requires_grad else functools.partial(_rhs64, b)
    r0 = lean(u, v, w)
    r1 = lean(u + dt * r0[0], _wall(v + dt * r0[1]), w + dt * r0[2])
    u, v, w = (q + 0.5 * dt * (x + y) for q, x, y in zip((u, v, w), r0, r1))
    v = _wall(v)
    p = _Solve.apply(b, _divergence64(b, u, v, w) / dt)
    gv = torch.cat([(p[1:] - p[:-1]) / b.dyc, torch.zeros_like(p[:1])])
    return (u - dt * (p.roll(-1, 2) - p) / b.dx, v - dt * gv, w - dt * (p.roll(-1, 1) - p) / b.dz, p)


def exact(case, seed):
    c = case
    b, dt, op = _Box(c), _dt(c), c["op"]
    x = tuple(t.to(F64) for t in _inputs(c, seed))
    if op == "poisson":
        return _poisson64(b, x[0])
    if op == "step":
        out = _step64(b, dt, *x)
        return out if c["pressure"] else out[:3]
    if op == "loop":
        stats = torch.zeros(c["ny"], 6, dtype=F64, device="cuda")
        for k in range(c["steps"]):
            x = _step64(b, dt, *x)[:3]
            if c["stats"] and (k + 1) % c["stats"] == 0:
                stats += torch.stack([q.mean(dim=(1, 2)) for q in (*x, *(q * q for q in x))], dim=1)
        return (*x, stats)
    g = tuple(t.to(F64) for t in _cotangent(c, seed))
    if _points(c) > 1 << 28:  # the recorded forward pass would not fit
        return (*_step64(b, dt, *x)[:3], None, None, None)
    y = x = tuple(t.requires_grad_(True) for t in x)
    for _ in range(c["steps"]):
        y = _step64(b, dt, *y)[:3]
    grads = torch.autograd.grad(y, x, g)
    return (*(t.detach() for t in y), *grads)
