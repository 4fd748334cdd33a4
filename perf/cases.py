"""Timed workloads of the library: what its users have it do, over the range of
grids, precisions and options that the entry points take.

A case is one call of a public entry point (`Context.run_ee`, `run_lim`,
`phiv`, `run_ee_batch`) from a given field.  Keys:
    kind     "ee", "lim", "phiv" or "batch"
    dim, n   grid (n points per direction)
    width    interface parameter in grid cells: eps = width * h
    theta    EE2: the proposed step is theta m_max^2 / rho, rho = eps^2 (4 dim / h^2)^2
             (about the spectral radius of Ahat; steps of theta above ~1/2 are
             shortened by the residual-time trace, smaller ones converge)
    order    LIM: the step is chosen so that the Chebyshev order is about this
    steps    accepted steps of the call
    fp32     FP32-mixed instead of FP64 (EE2)
    bc       "periodic" or "neumann" (the paper's domain (0, 64)^2)
    mobility variable mobility M(c) = 0.1 + (1 - c^2)
    field    "noise" (a quench: mean + small noise) or "grown" (separated
             phases with tanh interfaces, what a run spends its time on)

`exact` is the same mathematics in plain FP64 torch: modified Gram-Schmidt
Arnoldi with torch's matrix exponential, and the Chebyshev local iteration with
rolled arrays.
"""
import math

import numpy as np
import torch

from paper_2502_14589_amd import ch
from paper_2502_14589_amd.inputs import BATCH_SIDES

TOL = 1e-4
M_MAX = 30
MOBILITY = (0.1, 1.0)


def listed():
    return [
        # one step of the smallest workload, as a program that looks at every step calls it: latency
        {"name": "ee2 64sq fp64 step", "kind": "ee", "dim": 2, "n": 64, "width": 3.2, "theta": 0.1, "steps": 1, "m_max": 30,
         "fp32": False, "bc": "periodic", "mobility": False, "field": "noise"},
        # the paper's problem: Neumann boundaries, 128^2, adaptive EE2(30)
        {"name": "ee2 128sq neumann fp64", "kind": "ee", "dim": 2, "n": 128, "width": 1.92, "theta": 0.4, "steps": 6, "m_max": 30,
         "fp32": False, "bc": "neumann", "mobility": False, "field": "grown"},
        # an odd grid with variable mobility
        {"name": "ee2 333sq mobility fp64", "kind": "ee", "dim": 2, "n": 333, "width": 5.0, "theta": 0.4, "steps": 4, "m_max": 30,
         "fp32": False, "bc": "periodic", "mobility": True, "field": "grown"},
        # the flagship run in its two precisions: the steps of its long middle part (mostly shortened by the trace)
        {"name": "ee2 1024sq fp32", "kind": "ee", "dim": 2, "n": 1024, "width": 10.24, "theta": 0.9, "steps": 4, "m_max": 30,
         "fp32": True, "bc": "periodic", "mobility": False, "field": "grown"},
        {"name": "ee2 1024sq fp64", "kind": "ee", "dim": 2, "n": 1024, "width": 10.24, "theta": 0.4, "steps": 4, "m_max": 30,
         "fp32": False, "bc": "periodic", "mobility": False, "field": "grown"},
        # the largest 2-D grid in use
        {"name": "ee2 2048sq fp32", "kind": "ee", "dim": 2, "n": 2048, "width": 10.0, "theta": 0.4, "steps": 2, "m_max": 30,
         "fp32": True, "bc": "periodic", "mobility": False, "field": "grown"},
        # 3-D: an odd grid in FP64 and the 256^3 workload with its Krylov dimension 40
        {"name": "ee2 97cube fp64", "kind": "ee", "dim": 3, "n": 97, "width": 4.0, "theta": 0.2, "steps": 3, "m_max": 30,
         "fp32": False, "bc": "periodic", "mobility": False, "field": "grown"},
        {"name": "ee2 256cube fp32", "kind": "ee", "dim": 3, "n": 256, "width": 5.12, "theta": 0.03, "steps": 3, "m_max": 40,
         "fp32": True, "bc": "periodic", "mobility": False, "field": "grown"},
        # the local-iteration scheme (always FP64), 2-D and 3-D
        {"name": "lim 1024sq", "kind": "lim", "dim": 2, "n": 1024, "width": 10.24, "order": 200, "steps": 2, "bc": "periodic",
         "mobility": False, "field": "grown"},
        {"name": "lim 128cube", "kind": "lim", "dim": 3, "n": 128, "width": 4.0, "order": 40, "steps": 2, "bc": "periodic",
         "mobility": False, "field": "grown"},
        # the phi action alone with linear restarts, to a tight tolerance
        {"name": "phiv 300sq fp64", "kind": "phiv", "dim": 2, "n": 300, "width": 5.0, "theta": 2.0, "steps": 1, "m_max": 30,
         "fp32": False, "bc": "periodic", "mobility": False, "field": "grown"},
        # 64 ragged grids in one call (sides 128 to 512), FP32-mixed
        {"name": "batch 64 fp32", "kind": "batch", "dim": 2, "n": 64, "width": 0.0, "theta": 0.4, "steps": 3, "m_max": 30,
         "fp32": True, "bc": "periodic", "mobility": False, "field": "noise"},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case of the same ranges: 2-D sides 48..2048, 3-D sides 24..256, odd ones among them."""
    kind = rng.choice(["ee", "ee", "ee", "ee3", "lim", "lim3", "phiv", "batch"])
    dim = 3 if kind.endswith("3") else 2
    kind = kind.rstrip("3")
    if kind == "batch":
        return {"kind": "batch", "dim": 2, "n": rng.randint(4, 64), "width": 0.0, "theta": round(_log(rng, 0.1, 0.6), 3),
                "steps": rng.randint(1, 3), "m_max": 30, "fp32": rng.random() < 0.5, "bc": "periodic", "mobility": False,
                "field": "noise"}
    top = {("ee", 2): 2000, ("ee", 3): 230, ("lim", 2): 1400, ("lim", 3): 160, ("phiv", 2): 700}[(kind, dim)]
    n = int(_log(rng, 48 if dim == 2 else 24, top))
    if rng.random() < 0.5:
        n += n % 4 and 4 - n % 4
    bc, mob = "periodic", False
    if dim == 2:
        bc, mob = rng.choice([("periodic", False)] * 3 + [("neumann", False), ("periodic", True)])
    case = {"kind": kind, "dim": dim, "n": n, "width": round(rng.uniform(2.5, min(8.0, n / 12.0)), 2), "bc": bc, "mobility": mob,
            "field": rng.choice(["grown", "grown", "noise"])}
    if kind == "lim":
        return dict(case, order=int(_log(rng, 4, 200 if dim == 2 else 40)), steps=rng.randint(1, 2), field="grown")
    theta = {"ee": _log(rng, 0.02, 0.9), "phiv": rng.uniform(1.0, 2.5)}[kind]
    if dim == 3:
        theta = _log(rng, 0.01, 0.2)
    return dict(case, theta=round(theta, 4), steps=1 if kind == "phiv" else rng.randint(1, 4), m_max=rng.choice([12, 20, 30, 30, 40]),
                fp32=kind == "ee" and rng.random() < 0.5)


# -- inputs -----------------------------------------------------------------
class _Grid:
    """Plain numbers of a case's grid: length, h, eps, spectral radius, step."""

    def __init__(self, case, n=None, eps=None):
        self.dim, self.n, self.bc, self.mob = case["dim"], n or case["n"], case["bc"], case["mobility"]
        self.length = 64.0 if self.bc == "neumann" else 1.0
        self.h = self.length / self.n
        self.eps = eps or case["width"] * self.h
        self.rho = self.eps ** 2 * (4 * self.dim / self.h ** 2) ** 2
        if "theta" in case:
            self.tau = case["theta"] * case["m_max"] ** 2 / self.rho
        else:
            self.tau = (4.0 * case["order"] / math.pi) ** 2 / (1.1 * self.rho)
        self.shape = (self.n,) * self.dim


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _field(grid, kind, gen, mean):
    """A flat FP64 field on the grid, x fastest."""
    noise = torch.rand(grid.shape, generator=gen, device="cuda", dtype=torch.float64)
    if kind == "noise":
        return (mean + 0.1 * (noise - 0.5)).reshape(-1)
    if grid.bc == "neumann":   # even across the boundaries
        for d in range(grid.dim):
            noise = torch.cat([noise, noise.flip(d)], dim=d)
    # smooth over a few interface widths, then tanh interfaces of the model's width
    ell = 6.0 * grid.eps / grid.h
    for d in range(grid.dim):
        k = torch.fft.fftfreq(noise.shape[d], device="cuda", dtype=torch.float64) * 2 * math.pi * ell
        view = [1] * grid.dim
        view[d] = -1
        noise = torch.fft.ifft(torch.fft.fft(noise - 0.5 if d == 0 else noise, dim=d) * torch.exp(-0.5 * k * k).reshape(view), dim=d).real
    if grid.bc == "neumann":
        noise = noise[(slice(0, grid.n),) * grid.dim]
    g = noise / noise.square().mean().sqrt()
    return (0.97 * torch.tanh((g + mean) * (6.0 / math.sqrt(2.0)))).contiguous().reshape(-1)


def _problem(case, grid):
    return ch.Problem(grid.dim, grid.n, grid.eps, False, ch.CH_FP32_MIXED if case.get("fp32") else ch.CH_FP64,
                      ch.CH_BC_NEUMANN if grid.bc == "neumann" else ch.CH_BC_PERIODIC, grid.length,
                      MOBILITY if grid.mob else None)


def _members(case, seed):
    """Sides, grids and means of a batch: the sides of the ragged workload, eps log-uniform in [0.01, 0.05]."""
    rng = np.random.default_rng(int(seed))
    sides = rng.permutation(np.resize(np.asarray(BATCH_SIDES), case["n"]))
    eps = np.exp(rng.uniform(math.log(0.01), math.log(0.05), size=case["n"]))
    means = rng.uniform(-0.3, 0.3, size=case["n"])
    return [(_Grid(case, int(s), float(e)), float(m)) for s, e, m in zip(sides, eps, means)]


def _start(case, seed):
    gen = _generator(seed)
    if case["kind"] == "batch":
        grids = _members(case, seed)
        return [g for g, _ in grids], [_field(g, case["field"], gen, m) for g, m in grids]
    grid = _Grid(case)
    return grid, _field(grid, case["field"], gen, 0.1)


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    s.ctx = ch.Context(0)
    s.grid, s.y0 = _start(case, seed)
    if case["kind"] == "batch":
        s.y0 = torch.cat(s.y0)              # the fields are slices of one array
        s.y = torch.empty_like(s.y0)
        at = np.cumsum([0] + [g.n ** 2 for g in s.grid])
        s.fields = [s.y[a:b] for a, b in zip(at[:-1], at[1:])]
        s.ns, s.eps, s.taus = [g.n for g in s.grid], [g.eps for g in s.grid], [g.tau for g in s.grid]
    else:
        s.problem = _problem(case, s.grid)
        s.y = torch.empty_like(s.y0)
    return s


def run(s):
    c = s.case
    if c["kind"] == "phiv":
        rec = s.ctx.phiv(s.problem, s.y0, s.y, s.grid.tau, mode=ch.CH_PHI_RESTART, tol_phi=1e-8, m_max=c["m_max"])
        return {"y": s.y, "tau": rec["tau"], "matvecs": rec["matvecs"]}
    s.y.copy_(s.y0)
    if c["kind"] == "batch":
        st, _ = s.ctx.run_ee_batch(s.fields, s.ns, s.eps, precision=ch.CH_FP32_MIXED if c["fp32"] else ch.CH_FP64, tau0=s.taus,
                                   max_steps=c["steps"], m_max=c["m_max"], tol=TOL)
        return {"y": s.y, "t": np.array([x["t"] for x in st]), "matvecs": np.array([x["matvecs"] for x in st])}
    if c["kind"] == "lim":   # steps of the given size
        st, _ = s.ctx.run_lim(s.problem, s.y, s.grid.tau, max_steps=c["steps"], tol=0.0)
    else:
        st, _ = s.ctx.run_ee(s.problem, s.y, s.grid.tau, max_steps=c["steps"], m_max=c["m_max"], tol=TOL)
    return {"y": s.y, "t": st["t"], "matvecs": st["matvecs"]}


# -- the work of a pass -------------------------------------------------------
def _ee_work(points, dim, word, j, steps):
    """j Arnoldi iterations per step: iteration k orthogonalises against k columns (read once), reads its vector and the
    state and writes the next column; then the update and the estimate of the step.  Flops: two stencils, and a dot product
    and an axpy per column of each of the two Gram-Schmidt passes."""
    columns = j * (j - 1) / 2.0
    per_point = word * (columns + 3.0 * j) + word * j + 48.0
    flops = 8.0 * columns + j * (12.0 * dim + 20.0) + 2.0 * j + 60.0
    return {"bytes": points * per_point * steps, "flops": points * flops * steps}


def work(case):
    if case["kind"] == "lim":   # 2p - 1 stages, each reading two fields and writing one
        points = float(case["n"]) ** case["dim"]
        stages = (2 * case["order"] - 1) * case["steps"]
        return {"bytes": points * 24.0 * stages, "flops": points * (12.0 * case["dim"] + 25.0) * stages}
    # Krylov dimensions grow with the square root of the step until they reach m_max
    j = min(case["m_max"], 4 + 1.25 * case["m_max"] * math.sqrt(case["theta"]))
    word = 4.0 if case.get("fp32") else 8.0
    if case["kind"] == "batch":
        points = float(sum(int(s) ** 2 for s in np.resize(np.asarray(BATCH_SIDES), case["n"])))
        return _ee_work(points, 2, word, j, case["steps"])
    cycles = 1.0 + 4.0 * case["theta"] if case["kind"] == "phiv" else float(case["steps"])
    return _ee_work(float(case["n"]) ** case["dim"], case["dim"], word, j, cycles)


# -- the same in 64 bits ----------------------------------------------------------
class _Plain:
    """The discretised operators as plain torch expressions on one frozen state."""

    def __init__(self, grid):
        self.g = grid

    def _shift(self, v, d, by):
        if self.g.bc == "neumann":
            i = (torch.arange(self.g.n, device=v.device) + by).clamp(0, self.g.n - 1)
            return v.index_select(d, i)
        return torch.roll(v, -by, d)

    def lap(self, v):
        out = 2.0 * self.g.dim * v
        for d in range(self.g.dim):
            out = out - self._shift(v, d, 1) - self._shift(v, d, -1)
        return out / self.g.h ** 2

    def outer(self, v, y):
        if not self.g.mob:
            return self.lap(v)
        m = (MOBILITY[0] + MOBILITY[1] * (1.0 - y * y)).clamp(min=0.0)
        out = torch.zeros_like(v)
        for d in range(self.g.dim):
            for by in (1, -1):
                out = out + 0.5 * (m + self._shift(m, d, by)) * (v - self._shift(v, d, by))
        return out / self.g.h ** 2

    def f(self, y):
        return -self.outer(y ** 3 - y + self.g.eps ** 2 * self.lap(y), y)

    def jac(self, v, y):
        return self.outer((3.0 * y * y - 1.0) * v + self.g.eps ** 2 * self.lap(v), y)

    def ghat(self, y):
        return self.outer(2.0 * y ** 3, y)


def _small_phi(H, j, s):
    """s phi(-s H_jj) e_1 from the exponential of the augmented matrix."""
    X = torch.zeros(j + 1, j + 1, dtype=torch.float64)
    X[:j, :j] = -s * H[:j, :j]
    X[0, j] = s
    return torch.linalg.matrix_exp(X)[:j, j]


def _cycle(op, y, z, v, tau, tol, m):
    """One Krylov cycle from the state z with start vector v: (new state, covered step, dimension, converged)."""
    beta = float(v.norm())
    V = torch.empty(m + 1, v.numel(), dtype=torch.float64, device=v.device)
    H = torch.zeros(m + 1, m, dtype=torch.float64)
    V[0] = v.reshape(-1) / beta
    done = False
    for k in range(m):
        w = op.jac(V[k].reshape(y.shape), y).reshape(-1)
        for _ in range(2):
            c = V[:k + 1] @ w
            w = w - c @ V[:k + 1]
            H[:k + 1, k] += c.cpu()
        H[k + 1, k] = float(w.norm())
        V[k + 1] = w / H[k + 1, k]
        j, hn = k + 1, float(H[k + 1, k])
        u = _small_phi(H, j, tau)
        done = hn * abs(float(u[j - 1])) <= tol
        if done:
            break
    s = tau
    if not done:   # the largest step that passes: dyadic bracket, then bisection
        ok = lambda x: hn * abs(float(_small_phi(H, j, x)[j - 1])) <= tol  # noqa: E731
        lo = 0.5 * tau
        while not ok(lo):
            lo *= 0.5
        hi = 2.0 * lo
        for _ in range(50):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if ok(mid) else (lo, mid)
        s = lo
        u = _small_phi(H, j, s)
    znew = z + (beta * (u.to(v.device) @ V[:j])).reshape(y.shape)
    return znew, s, j, done


def _exact_ee(case, grid, y):
    op = _Plain(grid)
    y = y.reshape(grid.shape)
    tau, t, products = grid.tau, 0.0, 0
    f = op.f(y)
    for _ in range(case["steps"]):
        first = float(op.ghat(y).norm() / (10.0 * f.norm()))
        tol = max(min(first, 0.1, 10.0 * TOL), 1e-7)
        new, tau, j, _ = _cycle(op, y, y, f, tau, tol, case["m_max"])
        fnew = op.f(new)
        pc = y + 0.5 * tau * (f + fnew)
        est = float((new - pc).norm() / pc.norm())
        t += tau
        products += 1 + j
        tau = min(1.25 * tau, math.sqrt(TOL / est) * tau)
        y, f = new, fnew
    return y.reshape(-1), t, products


def _leja(p):
    beta = np.cos(np.pi * (2 * np.arange(p) + 1) / (2 * p))
    order, score = [0], np.zeros(p)
    for _ in range(p - 1):
        with np.errstate(divide="ignore"):
            score += np.log(np.abs(beta - beta[order[-1]]))
        top = score.max()
        order.append(int(np.flatnonzero(score >= top - 1e-9 * max(1.0, abs(top)))[0]))
    return order, beta


def _lambda_max(grid, y):
    """The largest absolute column sum of Ahat on a periodic grid with constant mobility."""
    a, d = 1.0 / grid.h ** 2, grid.dim
    e = grid.eps ** 2 * a * a
    c0, c1, rest = (20.0, 8.0, 12.0) if d == 2 else (42.0, 12.0, 30.0)
    q = y * y
    return max(abs(2 * d * x * a + c0 * e) + 2 * d * abs(x * a + c1 * e) + rest * e
               for x in (3.0 * float(q.min()) - 1.0, 3.0 * float(q.max()) - 1.0))


def _exact_lim(case, grid, y):
    op = _Plain(grid)
    y = y.reshape(grid.shape)
    tau, t, products = grid.tau, 0.0, 0
    for _ in range(case["steps"]):
        lam = _lambda_max(grid, y)
        p = math.ceil((math.pi / 4) / (math.pi / 2 - math.atan(math.sqrt(tau * lam))))
        order, beta = _leja(p)
        c, z = op.ghat(y), y
        for i in order + order[1:]:
            a = tau * lam / (1.0 + beta[0]) * (beta[0] - beta[i])
            z = (y + a * z + tau * (c - op.jac(z, y))) / (1.0 + a)
        y = z
        t += tau
        products += 2 * p - 1
    return y.reshape(-1), t, products


def exact(case, seed):
    grid, y = _start(case, seed)
    if case["kind"] == "batch":
        got = [_exact_ee(case, g, f) for g, f in zip(grid, y)]
        return {"y": torch.cat([x[0] for x in got]), "t": np.array([x[1] for x in got]), "matvecs": None}
    if case["kind"] == "lim":
        if grid.mob or grid.bc != "periodic":
            return None   # the bound of the spectrum has no short closed form there
        out, t, _ = _exact_lim(case, grid, y)
        return {"y": out, "t": t, "matvecs": None}
    if case["kind"] == "phiv":   # linear restarts: the residual of the frozen problem starts each cycle
        op = _Plain(grid)
        y = y.reshape(grid.shape)
        z, left = y, grid.tau
        while True:
            v = op.f(y) if z is y else op.ghat(y) - op.jac(z, y)
            z, s, _, done = _cycle(op, y, z, v, left, 1e-8, case["m_max"])
            if done:
                return {"y": z.reshape(-1), "tau": grid.tau, "matvecs": None}
            left -= s
    out, t, _ = _exact_ee(case, grid, y)
    return {"y": out, "t": t, "matvecs": None}
