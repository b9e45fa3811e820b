"""The calls whose speed this library is judged by, as a program of its users
makes them: short runs of the solver contexts (set the initial state, advance,
read the fields), the batched launch, the decomposed domain, the
three-dimensional scheme and the training step of the learned coefficient.

``listed()`` and ``draw()`` give cases (plain dicts), ``prepare()`` what a
program holds before the call, ``run()`` the call, ``work()`` the bytes and
operations it cannot do without, and ``exact()`` the same outputs from plain
torch in 64 bits: the scheme written out with whole-array operations, in the
textbook order, sharing nothing with the library.
"""

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1710_06423_amd import FP32, FP64, Batch, DecomposedSolver, Solver, even_cuts
from paper_1710_06423_amd.sacx3 import Solver3
from paper_1710_06423_amd.surrogate import Network

PERIODIC, OPEN = 0, 1
C2 = (0.02, 0.02, 0.2, 0.02)        # hyper-diffusion constants (density, thermal energy, velocity, field)
CSHK = (0.5, 0.5, 0.5, 0.5)
CFL = 0.3
DEV = "cuda"


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the paper's shock tube, at its 800 points: nothing but launches and latency
        dict(name="tube 800", kind="box", problem="tube", nx=800, ny=1, steps=40, fp32=False, hd=True),
        # a small box with odd sides, as in the smoke run and the tests
        dict(name="vortex 300x136", kind="box", problem="vortex", nx=300, ny=136, steps=20, fp32=False, hd=True),
        # the paper's middle size: the Orszag-Tang vortex at 1024^2
        dict(name="vortex 1024", kind="box", problem="vortex", nx=1024, ny=1024, steps=10, fp32=False, hd=True),
        # the headline size of the benchmark, far beyond every cache
        dict(name="vortex 8000", kind="box", problem="vortex", nx=8000, ny=8000, steps=2, fp32=False, hd=True),
        # FP32 bulk arithmetic
        dict(name="vortex 2048 fp32", kind="box", problem="vortex", nx=2048, ny=2048, steps=10, fp32=True, hd=True),
        # the paper's column without hyper-diffusion; open sides, sides that fit no tile
        dict(name="smooth 1501x997 no hd", kind="box", problem="smooth", nx=1501, ny=997, steps=10, fp32=False,
             hd=False),
        # a gravitationally stratified background, what the code exists for
        dict(name="atmosphere 1500x2000", kind="box", problem="atmosphere", nx=1500, ny=2000, steps=5, fp32=False,
             hd=True),
        # many small problems in one launch (tubes and boxes of the benchmark's ranges)
        dict(name="batch 8+8", kind="batch", tubes=8, boxes=8, steps=20, draw=3),
        # the paper's 2x2 split with halo exchange before every stage
        dict(name="domain 1024 2x2", kind="domain", nx=1024, ny=1024, px=2, py=2, steps=5),
        # three dimensions: a box that no cache holds, and a small ragged one with open sides
        dict(name="vortex3 256", kind="box3", problem="vortex", nx=256, ny=256, nz=256, steps=2, hd=True),
        dict(name="smooth3 75x53x61 open", kind="box3", problem="smooth", nx=75, ny=53, nz=61, steps=5, hd=True),
        # one training step of the learned coefficient on eight snapshots
        dict(name="train 8x256", kind="train", n=8, h=256, w=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["box", "box", "box", "box", "batch", "domain", "box3", "box3", "train"])
    if kind == "box":
        problem = rng.choice(["tube", "vortex", "vortex", "smooth", "atmosphere"])
        if problem == "tube":
            return dict(kind=kind, problem=problem, nx=_log(rng, 400, 3200), ny=1, steps=rng.randint(10, 40),
                        fp32=rng.random() < 0.3, hd=True)
        nx, ny = _log(rng, 64, 4000), _log(rng, 64, 4000)
        return dict(kind=kind, problem=problem, nx=nx, ny=ny, steps=max(1, min(20, 20000000 // (nx * ny))),
                    fp32=problem != "atmosphere" and rng.random() < 0.3, hd=problem != "smooth")
    if kind == "batch":
        return dict(kind=kind, tubes=rng.randint(0, 12), boxes=rng.randint(2, 12), steps=rng.randint(5, 20),
                    draw=rng.randint(0, 1 << 20))
    if kind == "domain":
        return dict(kind=kind, nx=_log(rng, 128, 1500), ny=_log(rng, 128, 1500), px=rng.randint(1, 3),
                    py=rng.randint(2, 3), steps=rng.randint(2, 8))
    if kind == "box3":
        nx, ny, nz = _log(rng, 24, 250), _log(rng, 24, 250), _log(rng, 24, 250)
        return dict(kind=kind, problem=rng.choice(["vortex", "smooth"]), nx=nx, ny=ny, nz=nz,
                    steps=max(1, min(10, 20000000 // (nx * ny * nz))), hd=rng.random() < 0.75)
    side = _log(rng, 64, 512)
    return dict(kind=kind, n=max(1, min(rng.randint(1, 8), (1 << 19) // (side * side))), h=side,
                w=max(32, min(512, side + rng.randint(-9, 9))))


# ---------------------------------------------------------------- inputs
def _rng(seed):
    return np.random.default_rng(int(seed))


def _centres(n, a, b):
    return a + (torch.arange(n, dtype=torch.float64, device=DEV) + 0.5) * ((b - a) / n)


def _fields(rho, v, p, b, gamma, shape):
    """Conserved fields from primitive ones: density, momenta, energy, field components."""
    full = lambda a: torch.as_tensor(a, dtype=torch.float64, device=DEV).expand(shape)  # noqa: E731
    rho, p = full(rho), full(p)
    v, b = [full(a) for a in v], [full(a) for a in b]
    e = p / (gamma - 1.0) + 0.5 * rho * sum(a * a for a in v) + 0.5 * sum(a * a for a in b)
    return torch.stack([rho] + [rho * a for a in v] + [e] + b)


def _modes(g, coords, shape, modes=4):
    """A smooth random field: a few Fourier modes over the unit box."""
    out = torch.zeros(shape, dtype=torch.float64, device=DEV)
    for _ in range(modes):
        k = g.integers(0, 4, size=len(coords))
        arg = sum(2.0 * math.pi * float(kk) * c for kk, c in zip(k, coords)) + float(g.uniform(0.0, 2.0 * math.pi))
        out = out + float(g.normal()) * torch.cos(arg)
    return out / modes


def _vortex(nx, ny, g):
    """Orszag-Tang on [0, 2 pi]^2: random field strength, random origin."""
    b0 = float(g.uniform(0.5, 1.5)) / math.sqrt(4.0 * math.pi)
    x = _centres(nx, 0.0, 2.0 * math.pi)[None, :] + float(g.uniform(0.0, 6.0))
    y = _centres(ny, 0.0, 2.0 * math.pi)[:, None] + float(g.uniform(0.0, 6.0))
    f = _fields(25.0 / (36.0 * math.pi), (-torch.sin(y), torch.sin(x)), 5.0 / (12.0 * math.pi),
                (-b0 * torch.sin(y), b0 * torch.sin(2.0 * x)), 5.0 / 3.0, (ny, nx))
    return SimpleNamespace(nx=nx, ny=ny, x0=0.0, x1=2.0 * math.pi, y0=0.0, y1=2.0 * math.pi, gamma=5.0 / 3.0,
                           bc=(PERIODIC,) * 4, fields=f, background=None, g=(0.0, 0.0), t0=0.0)


def _tube(n, g):
    """Brio-Wu on [0, 1], open ends: density and pressure of each side scaled."""
    sl, sr = float(g.uniform(0.5, 2.0)), float(g.uniform(0.5, 2.0))
    left = (_centres(n, 0.0, 1.0) < 0.5)[None, :]
    pick = lambda a, b: torch.where(left, torch.full_like(left, a, dtype=torch.float64),  # noqa: E731
                                    torch.full_like(left, b, dtype=torch.float64))
    f = _fields(pick(sl, 0.125 * sr), (0.0, 0.0), pick(sl, 0.1 * sr), (0.75, pick(1.0, -1.0)), 2.0, (1, n))
    return SimpleNamespace(nx=n, ny=1, x0=0.0, x1=1.0, y0=0.0, y1=1.0 / n, gamma=2.0,
                           bc=(OPEN, OPEN, PERIODIC, PERIODIC), fields=f, background=None, g=(0.0, 0.0), t0=0.0)


def _smooth(nx, ny, g):
    """A smooth random state with one pair of sides open."""
    c = (_centres(nx, 0.0, 1.0)[None, :], _centres(ny, 0.0, 1.0)[:, None])
    m = lambda: _modes(g, c, (ny, nx))  # noqa: E731
    f = _fields(1.0 + 0.2 * torch.tanh(m()), (0.5 * m(), 0.5 * m()), 1.0 + 0.2 * torch.tanh(m()),
                (0.5 * m(), 0.5 * m()), 5.0 / 3.0, (ny, nx))
    return SimpleNamespace(nx=nx, ny=ny, x0=0.0, x1=1.0, y0=0.0, y1=1.0, gamma=5.0 / 3.0,
                           bc=(OPEN, OPEN, PERIODIC, PERIODIC), fields=f, background=None, g=(0.0, 0.0), t0=0.0)


def _atmosphere(nx, ny, g):
    """An isothermal atmosphere under gravity with a wave pulse, x periodic, y open."""
    h, b_b = 0.25, (0.1, 0.2)
    x, y = _centres(nx, 0.0, 1.0)[None, :], _centres(ny, 0.0, 1.0)[:, None]
    rho_b = torch.exp(-y / h).expand(ny, nx)
    r2 = ((x - float(g.uniform(0.3, 0.7))) ** 2 + (y - float(g.uniform(0.15, 0.5))) ** 2) / 0.05 ** 2
    vy = 0.02 * math.sqrt(5.0 / 3.0 * h) * torch.exp(-r2)
    zero = torch.zeros(ny, nx, dtype=torch.float64, device=DEV)
    f = torch.stack([zero, zero, rho_b * vy, 0.5 * rho_b * vy * vy, zero, zero])
    bg = torch.stack([rho_b, rho_b * h / (2.0 / 3.0) + 0.5 * (b_b[0] ** 2 + b_b[1] ** 2),
                      torch.full_like(zero, b_b[0]), torch.full_like(zero, b_b[1])])
    return SimpleNamespace(nx=nx, ny=ny, x0=0.0, x1=1.0, y0=0.0, y1=1.0, gamma=5.0 / 3.0,
                           bc=(PERIODIC, PERIODIC, OPEN, OPEN), fields=f, background=bg, g=(0.0, -1.0), t0=0.0)


def _problem(case, seed):
    g = _rng(seed)
    if case["problem"] == "tube":
        return _tube(case["nx"], g)
    return {"vortex": _vortex, "smooth": _smooth, "atmosphere": _atmosphere}[case["problem"]](case["nx"], case["ny"], g)


def _problem3(case, seed):
    g, (nx, ny, nz) = _rng(seed), (case["nx"], case["ny"], case["nz"])
    shape = (nz, ny, nx)
    if case["problem"] == "vortex":   # the vortex carried into z, periodic
        ext, bc = (0.0, 2.0 * math.pi) * 3, (PERIODIC,) * 6
        x = _centres(nx, 0.0, ext[1])[None, None, :] + float(g.uniform(0.0, 6.0))
        y = _centres(ny, 0.0, ext[1])[None, :, None] + float(g.uniform(0.0, 6.0))
        z = _centres(nz, 0.0, ext[1])[:, None, None]
        b0, eps = float(g.uniform(0.5, 1.5)) / math.sqrt(4.0 * math.pi), 0.2
        mod = 1.0 + eps * torch.sin(z)
        f = _fields(25.0 / (36.0 * math.pi), (-mod * torch.sin(y), mod * torch.sin(x), eps * torch.sin(z)),
                    5.0 / (12.0 * math.pi), (-b0 * torch.sin(y), b0 * torch.sin(2.0 * x), 0.0), 5.0 / 3.0, shape)
    else:
        ext, bc = (0.0, 1.0) * 3, (OPEN, OPEN, PERIODIC, PERIODIC, OPEN, OPEN)
        c = (_centres(nx, 0.0, 1.0)[None, None, :], _centres(ny, 0.0, 1.0)[None, :, None],
             _centres(nz, 0.0, 1.0)[:, None, None])
        m = lambda: _modes(g, c, shape)  # noqa: E731
        f = _fields(1.0 + 0.2 * torch.tanh(m()), (0.5 * m(), 0.5 * m(), 0.5 * m()), 1.0 + 0.2 * torch.tanh(m()),
                    (0.5 * m(), 0.5 * m(), 0.5 * m()), 5.0 / 3.0, shape)
    return SimpleNamespace(nx=nx, ny=ny, nz=nz, extent=ext, gamma=5.0 / 3.0, bc=bc, fields=f, t0=0.0)


def _batch(case, seed):
    """The batch's sizes come with the case, its states from the seed."""
    sizes, g = _rng(case["draw"]), _rng(seed)
    out = [_tube(int(sizes.integers(400, 3201)), g) for _ in range(case["tubes"])]
    for _ in range(case["boxes"]):
        side = int(sizes.integers(128, 769))
        out.append(_vortex(side, side, g))
    return out


LAYERS = ((6, 32), (32, 32), (32, 32), (32, 10))
LR = 2e-3


def _training(case, seed):
    """Parameters, inputs, targets and weights of one training step: He-scaled
    weights, smooth normalised inputs, ratios mostly near 0, flux weights."""
    n, h, w = case["n"], case["h"], case["w"]
    gen = torch.Generator(device="cpu").manual_seed(int(seed))
    parts = []
    for l, (ci, co) in enumerate(LAYERS):
        parts.append(torch.randn(co * ci * 9, generator=gen) * math.sqrt(2.0 / (9 * ci)))
        parts.append(0.1 * torch.randn(co, generator=gen) - (2.0 if l == 3 else 0.0))
    theta = torch.cat(parts).to(DEV)
    g = _rng(seed)
    c = (_centres(w, 0.0, 1.0)[None, :], _centres(h, 0.0, 1.0)[:, None])
    x = torch.zeros(n, h, w, 8, dtype=torch.float64, device=DEV)
    for i in range(n):
        for k in range(6):
            x[i, :, :, k] = 3.0 * _modes(g, c, (h, w))
    dev = torch.Generator(device=DEV).manual_seed(int(seed))
    y = 4.0 * torch.rand((n, 10, h, w), generator=dev, device=DEV) ** 4
    wt = torch.rand((n, 10, h, w), generator=dev, device=DEV) ** 2
    return theta, x.to(torch.bfloat16), y, wt


# ---------------------------------------------------------------- prepare and run
def _precision(case):
    return FP32 if case.get("fp32") else FP64


def prepare(case, seed):
    kind = case["kind"]
    if kind == "box":
        p = _problem(case, seed)
        s = Solver.from_problem(p, precision=_precision(case), cfl=CFL, hd_on=case["hd"], init=False)
        return dict(kind=kind, solver=s, fields=p.fields, background=p.background, steps=case["steps"],
                    dtype=torch.float32 if case["fp32"] else torch.float64)
    if kind == "box3":
        p = _problem3(case, seed)
        return dict(kind=kind, solver=Solver3.from_problem(p, cfl=CFL, hd_on=case["hd"], init=False), fields=p.fields,
                    steps=case["steps"])
    if kind == "batch":
        ps = _batch(case, seed)
        return dict(kind=kind, batch=Batch(ps, precision=FP32, cfl=CFL, init=False), fields=[p.fields for p in ps],
                    steps=case["steps"])
    if kind == "domain":
        p = _vortex(case["nx"], case["ny"], _rng(seed))
        host = {k: p.fields[i].cpu().numpy() for i, k in enumerate(("rho", "mx", "my", "e", "bx", "by"))}
        xc, yc = even_cuts(case["nx"], case["px"]), even_cuts(case["ny"], case["py"])
        d = DecomposedSolver(SimpleNamespace(**{**vars(p), "fields": host}), xc, yc, cfl=CFL)
        parts = [[p.fields[:, yc[b]:yc[b + 1], xc[a]:xc[a + 1]].contiguous() for a in range(case["px"])]
                 for b in range(case["py"])]
        return dict(kind=kind, domain=d, parts=parts, steps=case["steps"])
    theta, x, y, wt = _training(case, seed)
    return dict(kind=kind, net=Network(theta=theta), x=x, y=y, wt=wt)


def run(state):
    """One run from its initial state to its fields (or one training step)."""
    kind = state["kind"]
    if kind == "box":
        s = state["solver"]
        s.init_state(state["fields"], state["background"])
        done, t = s.advance(state["steps"])
        return dict(u=s.read_fields(state["dtype"]), t=t, done=done)
    if kind == "box3":
        s = state["solver"]
        s.init_state(state["fields"])
        done, t = s.advance(state["steps"])
        return dict(u=s.read_fields(), t=t, done=done)
    if kind == "batch":
        b = state["batch"]
        for i, f in enumerate(state["fields"]):
            b[i].init_state(f)
        b.advance(state["steps"])
        return [b[i].read_fields(torch.float32) for i in range(len(b))]
    if kind == "domain":
        d = state["domain"]
        for row, parts in zip(d.subs, state["parts"]):
            for s, f in zip(row, parts):
                s.init_state(f)
        d.advance(state["steps"])
        return d.read_fields()
    net = state["net"]
    loss = net.train_step(state["x"], state["y"], LR, state["wt"])
    return dict(loss=loss, grad=net.grad, theta=net.theta, m=net.m, v=net.v)


# ---------------------------------------------------------------- work
# Operations per cell and RK stage (adds, multiplies, maxima and divisions of
# the scheme's definition, each counted once).
OPS = {(2, True): 700.0, (2, False): 170.0, (3, True): 1800.0, (3, False): 330.0}


def _solver_work(cells, nf, nbg, item, io_item, steps, dims, hd):
    """The initial state in, the fields out, and per step the state (and the
    static background) read once and the new state written once: the time step
    is a maximum over the whole new state, so no two steps can share a pass."""
    state = cells * nf * item
    return dict(bytes=cells * (nf + nbg) * io_item + state + steps * (2 * state + cells * nbg * item) + state +
                cells * nf * (4 if item == 4 else 8), flops=4.0 * steps * cells * OPS[(dims, hd)])


def work(case):
    kind = case["kind"]
    if kind == "box":
        return _solver_work(case["nx"] * case["ny"], 6, 4 if case["problem"] == "atmosphere" else 0,
                            4 if case["fp32"] else 8, 8, case["steps"], 2, case["hd"])
    if kind == "box3":
        return _solver_work(case["nx"] * case["ny"] * case["nz"], 8, 0, 8, 8, case["steps"], 3, case["hd"])
    if kind == "batch":
        sizes = _rng(case["draw"])
        cells = sum(int(sizes.integers(400, 3201)) for _ in range(case["tubes"]))
        cells += sum(int(sizes.integers(128, 769)) ** 2 for _ in range(case["boxes"]))
        return _solver_work(cells, 6, 0, 4, 8, case["steps"], 2, True)
    if kind == "domain":
        return _solver_work(case["nx"] * case["ny"], 6, 0, 8, 8, case["steps"], 2, True)
    pix = case["n"] * case["h"] * case["w"]
    mac = sum(9 * ci * co for ci, co in LAYERS)
    back = sum(9 * ci * co for ci, co in LAYERS[1:])      # the first layer's input has no gradient
    par = sum(9 * ci * co + co for ci, co in LAYERS)
    return dict(bytes=pix * (16 + 40 + 40) + 28.0 * par, flops=2.0 * pix * (2 * mac + back))


# ---------------------------------------------------------------- the same in 64 bits
class _Scheme:
    """The scheme on whole padded arrays, D = 2 or 3 directions (direction d
    is array axis D - 1 - d), by its definition: split ideal MHD, fourth-order
    differences, hyper-diffusion, classic RK4."""

    def __init__(self, n, h, gamma, bc, hd, background=None, g=None):
        self.D, self.n, self.h, self.gamma, self.bc, self.hd = len(n), n, h, gamma, bc, hd
        self.g = g or (0.0,) * len(n)
        self.index = []
        for d in range(self.D):
            i = torch.arange(-3, n[d] + 3, device=DEV)
            lo = i % n[d] if bc[2 * d] == PERIODIC else i.clamp(0, n[d] - 1)
            self.index.append(lo)
        self.bg = None if background is None else self.pad(background)

    def pad(self, f):
        for d in range(self.D):
            f = f.index_select(f.dim() - 1 - d, self.index[d])
        return f

    def at(self, a, d, k):
        """a shifted so that position i holds a[i + k] along direction d."""
        return a if k == 0 else torch.roll(a, -k, dims=a.dim() - 1 - d)

    def d4(self, a, d):
        return (8.0 * (self.at(a, d, 1) - self.at(a, d, -1)) - (self.at(a, d, 2) - self.at(a, d, -2))) / (12.0 * self.h[d])

    def ratio(self, q, d):
        d1 = self.at(q, d, 1) - q
        d3 = (self.at(q, d, 2) - self.at(q, d, -1)) - 3.0 * d1
        a1, a3 = d1.abs(), d3.abs()
        num = torch.maximum(torch.maximum(self.at(a3, d, -1), a3), self.at(a3, d, 1))
        den = torch.maximum(torch.maximum(self.at(a1, d, -1), a1), self.at(a1, d, 1))
        den = torch.maximum(torch.maximum(den, self.at(a1, d, -2)), self.at(a1, d, 2))
        return torch.where(den > 0.0, num / den, torch.zeros_like(num)), d1

    def primitives(self, u, bg):
        D = self.D
        rt, m, et, b = u[0], u[1:1 + D], u[1 + D], u[2 + D:]
        rb, eb, bb = (0.0, 0.0, [0.0] * D) if bg is None else (bg[0], bg[1], bg[2:])
        rho = rb + rt
        v = [a / rho for a in m]
        kin = 0.5 * sum(a * c for a, c in zip(m, v))
        bbd = sum(a * c for a, c in zip(bb, b))
        b2, b2b = sum(a * a for a in b), sum(a * a for a in bb)
        pk = (self.gamma - 1.0) * (et - kin - bbd - 0.5 * b2)
        pkb = (self.gamma - 1.0) * (eb - 0.5 * b2b)
        return rho, v, [x + y for x, y in zip(bb, b)], pk, pk + 0.5 * b2 + bbd, pkb, pkb + 0.5 * b2b

    def speeds(self, u):
        """The maxima of |v_d| + c_f over the cells of an unpadded state."""
        inner = tuple(slice(3, -3) for _ in range(self.D))
        bg = None if self.bg is None else [b[inner] for b in self.bg]
        rho, v, bt, pk, _, pkb, _ = self.primitives(u, bg)
        cf = torch.sqrt((self.gamma * (pk + pkb) + sum(a * a for a in bt)) / rho)
        return [float((a.abs() + cf).max()) for a in v]

    def rhs(self, state, cmax):
        D = self.D
        u = self.pad(state)
        rho, v, bt, pk, pt, _, ptb = self.primitives(u, self.bg)
        m, et, b = u[1:1 + D], u[1 + D], u[2 + D:]
        eb, bb = (0.0, [0.0] * D) if self.bg is None else (self.bg[1], self.bg[2:])
        bvt, bvb = sum(x * y for x, y in zip(b, v)), sum(x * y for x, y in zip(bb, v))
        K = [torch.zeros_like(rho) for _ in range(2 + 2 * D)]
        for d in range(D):
            K[0] -= self.d4(m[d], d)
            for k in range(D):
                f = v[d] * m[k] - (b[d] * b[k] + b[d] * bb[k] + bb[d] * b[k])
                K[1 + k] -= self.d4(f + pt if k == d else f, d)
                if k != d:
                    K[2 + D + k] -= self.d4(v[d] * bt[k] - bt[d] * v[k], d)
            K[1 + D] -= self.d4(v[d] * (et + eb + pt) - b[d] * (bvt + bvb) - bb[d] * bvt, d)
        if self.bg is not None:
            for k in range(D):
                for l in range(D):
                    K[1 + D] += bb[k] * bb[l] * self.d4(v[l], k)
                K[1 + D] -= ptb * self.d4(v[k], k)
        for d in range(D):
            if self.g[d] != 0.0:
                K[1 + d] += u[0] * self.g[d]
                K[1 + D] += u[0] * self.g[d] * v[d]
        if self.hd:
            self.hyper(K, u, rho, v, bt, pk / (self.gamma - 1.0), cmax)
        inner = tuple(slice(3, -3) for _ in range(D))
        return torch.stack([k[inner] for k in K])

    def hyper(self, K, u, rho, v, bt, eps, cmax):
        D, b = self.D, u[2 + self.D:]
        s = torch.clamp(-sum((self.at(v[d], d, 1) - self.at(v[d], d, -1)) / (2.0 * self.h[d]) for d in range(D)), min=0.0)
        G = []
        for d in range(D):
            h, sf = self.h[d], torch.maximum(s, self.at(s, d, 1))
            sets = {"r": (u[0], 0), "e": (eps, 1)}
            sets.update({("v", k): (v[k], 2) for k in range(D)})
            sets.update({("b", k): (b[k], 3) for k in range(D) if k != d})
            G.append({})
            for key, (q, c) in sets.items():
                R, d1 = self.ratio(q, d)
                G[d][key] = (C2[c] * h * cmax * R + CSHK[c] * h * h * sf) * d1 / h
        for d in range(D):
            mean = lambda a: 0.5 * (a + self.at(a, d, 1))  # noqa: E731

            def around(g, k):   # the four k-faces around a d-face
                two = self.at(g, k, -1) + g
                return (two + self.at(two, d, 1)) / 4.0

            def add(f, flux):
                K[f] += (flux - self.at(flux, d, -1)) / self.h[d]

            rf, energy = mean(rho), G[d]["e"].clone()
            add(0, G[d]["r"])
            for k in range(D):
                if k == d:
                    tau = rf * G[d][("v", k)]
                else:
                    tau = 0.5 * rf * (G[d][("v", k)] + around(G[k][("v", d)], k))
                    hb = G[d][("b", k)] - around(G[k][("b", d)], k)
                    add(2 + D + k, hb)
                    energy += mean(bt[k]) * hb
                add(1 + k, tau)
                energy += mean(v[k]) * tau
            add(1 + D, energy)

    def advance(self, u, steps):
        t = 0.0
        for _ in range(steps):
            c = self.speeds(u)
            active = [d for d in range(self.D) if self.n[d] > 1]
            dt = CFL * min(self.h[d] / c[d] for d in active)
            cmax = max(c[d] for d in active)
            k1 = self.rhs(u, cmax)
            k2 = self.rhs(u + 0.5 * dt * k1, cmax)
            k3 = self.rhs(u + 0.5 * dt * k2, cmax)
            k4 = self.rhs(u + dt * k3, cmax)
            u = u + (dt / 6.0) * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
            t += dt
        return u, t


def _exact_box(p, steps, hd):
    s = _Scheme((p.nx, p.ny), ((p.x1 - p.x0) / p.nx, (p.y1 - p.y0) / p.ny), p.gamma, p.bc, hd, p.background, p.g)
    return s.advance(p.fields, steps)


def _exact_training(case, seed):
    """Forward with BF16 weights and activations, gradients, one Adam step from zero moments."""
    theta, x, y, wt = _training(case, seed)
    n, h, w = case["n"], case["h"], case["w"]
    bf = lambda a: a + (a.to(torch.bfloat16).double() - a).detach()  # noqa: E731
    th = theta.double().requires_grad_(True)
    a, o = x[..., :6].double(), 0
    for l, (ci, co) in enumerate(LAYERS):
        wk = bf(th[o:o + 9 * ci * co]).view(co, ci, 3, 3)
        bias = th[o + 9 * ci * co:o + 9 * ci * co + co]
        o += 9 * ci * co + co
        z = bias
        for dy in range(3):
            for dx in range(3):
                z = z + torch.roll(a, (1 - dy, 1 - dx), dims=(1, 2)).reshape(-1, ci) @ wk[:, :, dy, dx].t().contiguous()
        a = (4.0 * torch.sigmoid(z) if l == 3 else bf(torch.relu(z))).view(n, h, w, co)
    loss = (wt.double() * (a.permute(0, 3, 1, 2) - y.double()) ** 2).mean()
    grad, = torch.autograd.grad(loss, th)
    m, v = 0.1 * grad, 0.001 * grad * grad
    new = theta.double() - LR * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return dict(loss=loss.detach().view(1), grad=grad, theta=new, m=m, v=v)


def exact(case, seed):
    kind = case["kind"]
    if kind == "box":
        u, t = _exact_box(_problem(case, seed), case["steps"], case["hd"])
        return dict(u=u, t=t, done=None)
    if kind == "box3":
        p = _problem3(case, seed)
        e = p.extent
        h = tuple((e[2 * d + 1] - e[2 * d]) / k for d, k in enumerate((p.nx, p.ny, p.nz)))
        u, t = _Scheme((p.nx, p.ny, p.nz), h, p.gamma, p.bc, case["hd"]).advance(p.fields, case["steps"])
        return dict(u=u, t=t, done=None)
    if kind == "batch":
        return [_exact_box(p, case["steps"], True)[0] for p in _batch(case, seed)]
    if kind == "domain":
        return _exact_box(_vortex(case["nx"], case["ny"], _rng(seed)), case["steps"], True)[0]
    return _exact_training(case, seed)
