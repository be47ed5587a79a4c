"""Work that programs have this library do, for timing: solves of one problem, uniform and ragged batches,
gradients and served requests, each through the library's entry points.

A case is a dict of plain values; `kind` says how it is run:
  run     one context over `count` problems of `n` nodes, `steps` steps of `scheme`;
  mixed   one context over a ragged batch (n log-uniform in [n_lo, n_hi], half explicit and half BTCS, both
          boundary types): `steps` explicit and `btcs_steps` BTCS steps in one call;
  adjoint forward run, loss 1/2 |u_T - target|^2 and its gradients with respect to u0 and nu, with
          checkpoints every `ckpt` steps;
  serve   an explicit and a BTCS slot pool, `count` ragged requests each: admitted, ticked until done,
          retired.
Problems live on [0, 2 pi] (one long Dirichlet grid on [0, 1]) with nu ~ U[0.005, 0.1] and eight-mode
initial states 1 + sum (g_k / k) sin(k x), g_k ~ N(0, 1); Dirichlet values are 1.  Time steps are multiples
of the CFL step (eqs. 7-8 with factor 0.5): 1 for the explicit schemes, 10 for BTCS and Crank-Nicolson, 2
for Newton.
"""
import math
import types

import numpy as np
import torch

import paper_2601_12204_amd as B

SCHEMES = {"explicit": B.EXPLICIT, "btcs": B.BTCS, "rk4": B.RK4, "cn": B.CN, "newton": B.NEWTON}
FACTOR = {B.EXPLICIT: 1.0, B.RK4: 1.0, B.BTCS: 10.0, B.CN: 10.0, B.NEWTON: 2.0}
MODES = 8
SLOTS = 128                 # slots of a serving pool
POOL_NODES = 65536          # longest problem a pool holds
TICK = {B.EXPLICIT: 1000, B.BTCS: 100}


def listed():
    return [
        # One shock problem on the paper's small grid, explicit to t = 0.5: the latency of a single solve.
        dict(name="single_explicit", kind="run", scheme="explicit", bc="periodic", n=101, count=1, steps=113, dtype="f64"),
        # The same problem by BTCS at ten times the step.
        dict(name="single_btcs", kind="run", scheme="btcs", bc="periodic", n=101, count=1, steps=12, dtype="f64"),
        # A parameter sweep: thousands of equal grids advanced by forward Euler.
        dict(name="batch_explicit", kind="run", scheme="explicit", bc="periodic", n=8192, count=4096, steps=1000, dtype="f64"),
        # The same sweep by BTCS.
        dict(name="batch_btcs", kind="run", scheme="btcs", bc="periodic", n=8192, count=4096, steps=200, dtype="f64"),
        # The sweep with the paper's other integrators: RK4 in single precision, ...
        dict(name="batch_rk4_f32", kind="run", scheme="rk4", bc="periodic", n=8192, count=4096, steps=200, dtype="f32"),
        # ... Crank-Nicolson ...
        dict(name="batch_cn", kind="run", scheme="cn", bc="periodic", n=8192, count=4096, steps=100, dtype="f64"),
        # ... and the fully implicit step by Newton's method.
        dict(name="batch_newton", kind="run", scheme="newton", bc="periodic", n=8192, count=4096, steps=20, dtype="f64"),
        # One very fine grid with a viscous shock between fixed ends.
        dict(name="long_btcs", kind="run", scheme="btcs", bc="dirichlet", n=1 << 24, count=1, steps=128, dtype="f64"),
        # A study over many grids, boundary types and both schemes in one call.
        dict(name="ragged_mixed", kind="mixed", n_lo=64, n_hi=65536, count=10000, steps=1000, btcs_steps=100, dtype="f64"),
        # A burst of requests to the serving pools.
        dict(name="serve_f32", kind="serve", n_lo=64, n_hi=65536, count=64, steps=1000, btcs_steps=100, dtype="f32"),
        # Fitting initial states and viscosities to a later state, through the explicit step ...
        dict(name="grad_explicit", kind="adjoint", scheme="explicit", bc="periodic", n=16384, count=256, steps=1000, ckpt=100, dtype="f64"),
        # ... and through the BTCS step.
        dict(name="grad_btcs", kind="adjoint", scheme="btcs", bc="periodic", n=16384, count=256, steps=1000, ckpt=100, dtype="f64"),
    ]


def _spread(rng, lo, hi):
    """A whole number of [lo, hi], uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "run", "mixed", "adjoint", "serve"])
    dtype = rng.choice(["f64", "f64", "f32"])
    bc = rng.choice(["periodic", "dirichlet"])
    if kind == "mixed":
        return dict(kind=kind, n_lo=64, n_hi=_spread(rng, 1000, 65536), count=_spread(rng, 20, 4000),
                    steps=_spread(rng, 100, 1000), btcs_steps=_spread(rng, 10, 100), dtype=dtype)
    if kind == "serve":
        return dict(kind=kind, n_lo=64, n_hi=_spread(rng, 1000, 65536), count=_spread(rng, 1, SLOTS),
                    steps=1000, btcs_steps=100, dtype=dtype)
    if kind == "adjoint":
        scheme = rng.choice(["explicit", "btcs"])
        n = rng.choice([4096, 8192, 16384, _spread(rng, 64, 65536)])
        return dict(kind=kind, scheme=scheme, bc=bc, n=n, count=_spread(rng, 1, max(1, (1 << 21) // n)),
                    steps=_spread(rng, 20, 500 if scheme == "explicit" else 200), ckpt=rng.choice([10, 25, 50, 100]),
                    dtype="f64")
    scheme = rng.choice(sorted(SCHEMES))
    steps = {"explicit": (50, 1000), "btcs": (5, 200), "rk4": (20, 200), "cn": (5, 100), "newton": (2, 20)}[scheme]
    if scheme in ("explicit", "btcs") and rng.random() < 0.2:        # one long grid
        return dict(kind=kind, scheme=scheme, bc=bc, n=_spread(rng, 1 << 17, 1 << 24), count=1,
                    steps=_spread(rng, *steps) // 2 + 1, dtype=dtype)
    n = rng.choice([_spread(rng, 64, 65536), _spread(rng, 64, 8192), 1 << rng.randint(6, 13)])
    nodes = 1 << (22 if scheme == "newton" else 25)
    return dict(kind=kind, scheme=scheme, bc=bc, n=n, count=_spread(rng, 1, max(1, min(4096, nodes // n))),
                steps=_spread(rng, *steps), dtype=dtype)


# ---------------------------------------------------------------------------------------------- inputs
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _batch(case, seed, half=None):
    """Parameters and initial states of a case's problems: numpy arrays of one value per problem, and the
    packed binary64 states (instance starts aligned as the library's).  The seed gives nu and the initial
    states; a ragged case's sizes, boundary types and schemes are its own, alike for every seed.  `half`:
    the scheme of a serving pool's requests."""
    rng = np.random.default_rng([int(seed), 12204 + (half or 0)])
    mix = np.random.default_rng([12204 + (half or 0), int(case["count"])])
    count, dev = int(case["count"]), _device()
    nu = rng.uniform(0.005, 0.1, size=count)
    g = rng.standard_normal((count, MODES))
    if case["kind"] in ("mixed", "serve"):
        n = np.rint(np.exp(mix.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), size=count))).astype(np.int64)
        bc = mix.integers(0, 2, size=count)
        scheme = mix.integers(0, 2, size=count) if half is None else np.full(count, half)
    else:
        n = np.full(count, int(case["n"]), dtype=np.int64)
        bc = np.full(count, B.BC_DIRICHLET if case["bc"] == "dirichlet" else B.BC_PERIODIC)
        scheme = np.full(count, SCHEMES[case["scheme"]])
    long_grid = case["kind"] == "run" and case["n"] > 65536
    length = np.full(count, 1.0 if long_grid else 2.0 * math.pi)
    left = np.where(bc == B.BC_DIRICHLET, 1.0, 0.0)
    right = left.copy()
    if long_grid:
        nu = nu * 1e-2 / 5.0                          # about 1e-4: a thin layer on [0, 1]
        right[:] = 0.0
    padded = (n + B.ALIGN - 1) // B.ALIGN * B.ALIGN
    off = np.concatenate([[0], np.cumsum(padded)])
    inst = torch.repeat_interleave(torch.arange(count, device=dev), torch.from_numpy(padded).to(dev))
    j = torch.arange(int(off[-1]), device=dev) - torch.from_numpy(off[:-1]).to(dev)[inst]
    last = torch.from_numpy(n - 1).to(dev)[inst]
    real = j <= last
    dx = np.where(bc == B.BC_PERIODIC, length / n, length / (n - 1))
    x = j * torch.from_numpy(dx).to(dev)[inst]
    if long_grid:
        at = torch.from_numpy(0.3 + 0.02 * g[:, 0]).to(dev)[inst]
        u = 0.5 * (1.0 - torch.tanh((x - at) / 0.01))
    else:
        u = torch.ones_like(x)
        for k in range(MODES):
            u += torch.from_numpy(g[:, k] / (k + 1)).to(dev)[inst] * torch.sin((k + 1) * x)
    fixed = torch.from_numpy(bc == B.BC_DIRICHLET).to(dev)[inst]
    u = torch.where(fixed & (j == 0), torch.from_numpy(left).to(dev)[inst], u)
    u = torch.where(fixed & (j == last), torch.from_numpy(right).to(dev)[inst], u)
    u = torch.where(real, u, torch.zeros_like(u))
    if case["dtype"] == "f32":
        u = u.float().double()
    top = torch.zeros(count, dtype=torch.float64, device=dev).scatter_reduce_(0, inst, u.abs(), "amax").cpu().numpy()
    factor = np.array([FACTOR[int(s)] for s in scheme])
    with np.errstate(divide="ignore"):
        dt = factor * (0.5 * np.minimum(dx / top, dx * dx / (2.0 * nu)))
    return types.SimpleNamespace(n=n, bc=bc, scheme=scheme, length=length, nu=nu, left=left, right=right, dx=dx, dt=dt,
                                 off=off, u=u, inst=inst, j=j)


def _problems(b):
    return [types.SimpleNamespace(n=int(n), length=float(length), nu=float(nu), dt=float(dt), bc=int(bc), scheme=int(s),
                                  left=float(a), right=float(c))
            for n, length, nu, dt, bc, s, a, c in zip(b.n, b.length, b.nu, b.dt, b.bc, b.scheme, b.left, b.right)]


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _targets(case, seed):
    """The states a gradient case is fitted to: a second draw of initial states."""
    return _batch(case, seed + 104729).u


# ------------------------------------------------------------------------------------------- the cases
def prepare(case, seed):
    td = _dtype(case)
    if case["kind"] == "serve":
        halves = []
        for scheme in (B.EXPLICIT, B.BTCS):
            b = _batch(case, seed, half=scheme)
            u0 = b.u.to(td)
            stream = torch.cuda.Stream()
            pool = B.Pool(td, scheme, SLOTS, POOL_NODES, TICK[scheme], stream=stream.cuda_stream)
            word = u0.element_size()
            halves.append(types.SimpleNamespace(
                pool=pool, stream=stream, problems=_problems(b), u0=u0, out=torch.zeros_like(u0),
                src=[u0.data_ptr() + int(o) * word for o in b.off[:-1]],
                steps=case["steps"] if scheme == B.EXPLICIT else case["btcs_steps"]))
            halves[-1].dst = [halves[-1].out.data_ptr() + int(o) * word for o in b.off[:-1]]
        return types.SimpleNamespace(case=case, halves=halves)
    b = _batch(case, seed)
    solver = B.Solver(_problems(b), dtype=td)
    u0 = b.u.to(td)
    s = types.SimpleNamespace(case=case, solver=solver, u0=u0, u=torch.empty_like(u0))
    if case["kind"] == "adjoint":
        s.target = _targets(case, seed).to(td)
        s.grad_u0 = torch.zeros_like(u0)
        s.grad_nu = torch.zeros(solver.count, dtype=td, device=u0.device)
    return s


def run(s):
    case = s.case
    if case["kind"] == "serve":
        return _serve(s)
    s.u.copy_(s.u0)
    if case["kind"] == "mixed":
        s.solver.run_mixed(s.u, case["steps"], case["btcs_steps"])
        return s.u
    s.solver.run(s.u, case["steps"])
    if case["kind"] == "run":
        return s.u
    lam = s.u - s.target
    B.adjoint_into(s.solver, s.u0, lam, case["steps"], case["ckpt"], s.grad_u0, s.grad_nu)
    return {"u": s.u, "grad_u0": s.grad_u0, "grad_nu": s.grad_nu}


def _serve(s):
    now = torch.cuda.current_stream()
    slots = []
    for h in s.halves:
        h.stream.wait_stream(now)
        slots.append([h.pool.admit(p, src, h.steps) for p, src in zip(h.problems, h.src)])
    busy = True
    while busy:
        busy = False
        for h, own in zip(s.halves, slots):
            if any(h.pool.remaining(k) > 0 for k in own):
                h.pool.tick()
                busy = True
    for h, own in zip(s.halves, slots):
        for k, dst in zip(own, h.dst):
            h.pool.retire(k, dst)
        now.wait_stream(h.stream)
    return [h.out for h in s.halves]


# Operations of one node and step: the row's assembly and elimination for the implicit schemes.
FLOPS = {"explicit": 12, "btcs": 16, "rk4": 57, "cn": 18, "newton": 4 * 26}


def work(case):
    word = 4 if case["dtype"] == "f32" else 8
    if case["kind"] in ("run", "adjoint"):
        nodes = case["n"] * case["count"]
        flops = nodes * case["steps"] * FLOPS[case["scheme"]]
        if case["kind"] == "run":
            return {"bytes": 2 * word * nodes, "flops": flops}
        # u0 and the target read, u_T and the gradient written; the reverse sweep's transposed stencil or solve
        return {"bytes": 4 * word * nodes, "flops": flops + nodes * case["steps"] * 20}
    mean = (case["n_hi"] - case["n_lo"]) / math.log(case["n_hi"] / case["n_lo"])
    share = 0.5 if case["kind"] == "mixed" else 1.0                 # of `count`, for each of the two schemes
    nodes = mean * case["count"] * share
    return {"bytes": 2 * 2 * word * nodes,
            "flops": nodes * (case["steps"] * FLOPS["explicit"] + case["btcs_steps"] * FLOPS["btcs"])}


# ------------------------------------------------------------------- the same results in plain binary64
class _Grid:
    """Neighbour indices and per-node coefficients of packed problems."""

    def __init__(self, b, members):
        dev = b.u.device
        keep = np.zeros(len(b.n), dtype=bool)
        keep[members] = True
        n = torch.from_numpy(b.n).to(dev)
        self.at = torch.nonzero(torch.from_numpy(keep).to(dev)[b.inst] & (b.j < n[b.inst])).reshape(-1)
        inst, self.j = b.inst[self.at], b.j[self.at]
        own = np.where(keep, b.n, 0)
        self.base = torch.from_numpy(np.concatenate([[0], np.cumsum(own)])[:-1]).to(dev)[inst]
        self.n = n[inst]
        self.inst = inst

        def node(v):
            return torch.from_numpy(np.asarray(v, dtype=np.float64)).to(dev)[inst]

        self.r, self.D = node(b.dt / b.dx), node(b.nu * b.dt / (b.dx * b.dx))
        first, last = self.j == 0, self.j == self.n - 1
        fixed = torch.from_numpy(b.bc == B.BC_DIRICHLET).to(dev)[inst]
        self.end = fixed & (first | last)
        self.value = torch.where(first, node(b.left), node(b.right))
        self.any_end = bool(self.end.any())
        self.m, self.p = self.shift(-1), self.shift(1)

    def shift(self, s):
        return self.base + torch.remainder(self.j + s, self.n)

    def ends(self, u):
        return torch.where(self.end, self.value, u) if self.any_end else u

    def inner(self, v, other=0.0):
        return torch.where(self.end, torch.full_like(v, other), v) if self.any_end else v

    def rate(self, u):
        """dt times the explicit right-hand side (eq. 21); zero at fixed nodes."""
        c, um, up = self.r * u, u[self.m], u[self.p]
        k = self.D * ((up + um) - 2.0 * u) - (c.clamp(min=0) * (u - um) + c.clamp(max=0) * (up - u))
        return self.inner(k)

    def solve(self, a, d, c, y):
        """Tridiagonal systems (cyclic; fixed ends are rows of their own) by cyclic reduction."""
        a, c, y, s = a / d, c / d, y / d, 1
        while True:
            top = float((a.abs() + c.abs()).max())
            if top < 1e-19 or s >= int(self.n.max()) and bool((self.n & (self.n - 1) == 0).all()):
                return y / (1.0 + a + c) if s >= int(self.n.max()) else y
            m, p = self.shift(-s), self.shift(s)
            w = 1.0 / (1.0 - a * c[m] - c * a[p])
            a, c, y = -a * a[m] * w, -c * c[p] * w, (y - a * y[m] - c * y[p]) * w
            s *= 2

    def rows(self, u, h=1.0):
        c, D = h * self.r * u, h * self.D
        lo, up = -(D + c.clamp(min=0)), c.clamp(max=0) - D
        return self.inner(lo), self.inner((1.0 + 2.0 * D) + c.abs(), 1.0), self.inner(up)

    def step(self, u, scheme):
        if scheme == B.EXPLICIT:
            return u + self.rate(u)
        if scheme == B.RK4:
            k1 = self.rate(u)
            k2 = self.rate(u + 0.5 * k1)
            k3 = self.rate(u + 0.5 * k2)
            return u + (k1 + 2.0 * k2 + 2.0 * k3 + self.rate(u + k3)) / 6.0
        if scheme == B.BTCS:
            return self.solve(*self.rows(u), u)
        if scheme == B.CN:
            return 2.0 * self.solve(*self.rows(u, 0.5), u) - u
        x, h = u, 0.5 * self.r
        for _ in range(4):
            xm, xp = x[self.m], x[self.p]
            F = (x - u) + (h * x * (xp - xm) - self.D * ((xp + xm) - 2.0 * x))
            x = x + self.solve(self.inner(-h * x - self.D), self.inner((1.0 + 2.0 * self.D) + h * (xp - xm), 1.0),
                               self.inner(h * x - self.D), self.inner(-F))
        return x

    def advance(self, u, scheme, steps):
        u = self.ends(u)
        for _ in range(steps):
            u = self.step(u, scheme)
        return u

    def back(self, y, x, lam, scheme):
        """lam at step k from lam at k + 1, with y = u^k and x = u^(k+1), and dJ/dD per node."""
        lam = self.inner(lam)
        pos = y >= 0
        if scheme == B.EXPLICIT:
            ym, yp, r, D = y[self.m], y[self.p], self.r, self.D
            own = 1.0 - 2.0 * D - torch.where(pos, r * (y - ym) + r * y, r * (yp - y) - r * y)
            to_right = torch.where(pos, r * y + D, D)           # what row i takes from node i - 1
            to_left = torch.where(pos, D, D - r * y)            # ... and from node i + 1
            out = own * lam + (to_right * lam)[self.p] + (to_left * lam)[self.m]
            return self.inner(out), lam * ((yp + ym) - 2.0 * y)
        lo, d, up = self.rows(y)
        mu = self.inner(self.solve(self.inner(up[self.m]), d, self.inner(lo[self.p]), lam))
        xm, xp = x[self.m], x[self.p]
        G = torch.where(pos, self.r * (x - xm), self.r * (xp - x))
        return self.inner((1.0 - G) * mu), -mu * ((2.0 * x - xm) - xp)


def _cost(case):
    """About how many passes over a node the plain evaluation makes, in nodes."""
    per = {"explicit": 1, "rk4": 5, "btcs": 12, "cn": 12, "newton": 60}
    if case["kind"] in ("run", "adjoint"):
        nodes = case["n"] * case["count"] + 20000
        return nodes * case["steps"] * per[case["scheme"]] * (3 if case["kind"] == "adjoint" else 1)
    nodes = work(case)["bytes"] / (8 * (2 if case["dtype"] == "f32" else 4)) + 20000
    return nodes * (case["steps"] + 12 * case["btcs_steps"])


def exact(case, seed):
    if _cost(case) > (1.6e11 if torch.cuda.is_available() else 2e8):
        return None
    if case["kind"] == "adjoint" and case["n"] * case["count"] * case["steps"] * 8 > 6e10:
        return None
    if case["kind"] == "serve":
        out = []
        for scheme in (B.EXPLICIT, B.BTCS):
            out.append(_forward(_batch(case, seed, half=scheme), case))
        return out
    b = _batch(case, seed)
    if case["kind"] != "adjoint":
        return _forward(b, case)
    scheme = int(b.scheme[0])
    grid = _Grid(b, np.arange(len(b.n)))
    states = [b.u[grid.at]]
    for k in range(case["steps"]):
        states.append(grid.step(states[-1] if k else grid.ends(states[-1]), scheme))
    uT, u0 = b.u.clone(), torch.zeros_like(b.u)
    uT[grid.at] = states[-1]
    lam = (uT - _targets(case, seed))[grid.at]
    g = torch.zeros_like(lam)
    for k in range(case["steps"] - 1, -1, -1):
        x = states.pop()
        lam, part = grid.back(grid.ends(states[-1]), x, lam, scheme)
        g += part
    u0[grid.at] = lam
    nu = torch.zeros(len(b.n), dtype=torch.float64, device=lam.device).index_add_(0, grid.inst, grid.inner(g))
    return {"u": uT, "grad_u0": u0, "grad_nu": nu * torch.from_numpy(b.dt / (b.dx * b.dx)).to(lam.device)}


def _forward(b, case):
    out = b.u.clone()
    for scheme in sorted(set(int(s) for s in b.scheme)):
        grid = _Grid(b, np.nonzero(b.scheme == scheme)[0])
        steps = case["btcs_steps"] if "btcs_steps" in case and scheme == B.BTCS else case["steps"]
        out[grid.at] = grid.advance(b.u[grid.at], scheme, steps)
    return out
