"""Timing cases of the library: what its users run, each through a public entry point.

A case is a dict of plain values.  ``listed()`` gives the fixed ones, ``draw(rng)`` one more of
the same ranges, ``prepare(case, seed)`` what a user's program holds before the call (plan or
server, device fields), ``run(state)`` one pass, ``exact(case, seed)`` the same outputs from
dense 64-bit linear algebra (boxes only; a box operator is separable), ``work(case)`` the bytes
and operations one pass cannot do without.

Paths:
  solve       one Poisson solve (Plan.solve), FP64 or mixed, retiring or lockstep modes
  helmholtz   the implicit-diffusion solves of one Runge-Kutta step: three terms alpha, one plan
  project     one pressure projection of a predicted velocity (Plan.project)
  batch       many uneven boxes in one call (solve_batch)
  serve       a burst of requests through the serving loop (Server.submit / wait)
  mg3d        the 3D multigrid without the z synthesis (Plan3D.solve)
  transform   forward and inverse z transform alone (Plan.forward / inverse)
  operator    L_h p, the residual check and the divergence, as a program that composes its own
              time step calls them
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2106_03583_amd as mbp

D, N, C, P = mbp.DIRICHLET, mbp.NEUMANN, mbp.CONNECT, mbp.PERIODIC
PAIRS = {"PP": (P, P), "NN": (N, N), "DD": (D, D), "ND": (N, D), "DN": (D, N)}
KINDS = ["PP", "NN", "DD", "ND", "DN"]
H = 1.0 / 128.0  # cell width of the boxes before stretching
RTOL = 1e-10


def listed():
    box = lambda name, nx, ny, nz, pairs, **kw: dict(  # noqa: E731
        dict(name=name, path="solve", shape="box", nx=nx, ny=ny, nz=nz, pairs=pairs, stretch=0.0, precision="fp64",
             retire=True), **kw)
    return [
        # the smallest configuration: a unit box of 32^3, where launches and latency count
        box("solve_box_32", 32, 32, 32, "DD NN PP"),
        # an ordinary box with odd x-y counts, stretched walls, the default flags (lockstep modes)
        box("solve_box_odd_lockstep", 203, 157, 90, "ND DD NN", stretch=1.3, retire=False),
        # the three-block L-shaped duct, all walls Neumann (singular plane), periodic z
        dict(name="solve_lshape", path="solve", shape="lshape", n=256, nz=512, stretch=1.5, precision="fp64",
             retire=True),
        # the largest single problem: the 512 x 512 x 1024 box
        box("solve_box_512x512x1024", 512, 512, 1024, "DD NN NN"),
        # eight blocks around a square obstacle in mixed precision
        dict(name="solve_obstacle_mixed", path="solve", shape="obstacle", n=64, nz=576, stretch=0.0,
             precision="mixed", retire=True),
        # three implicit-diffusion substeps on a duct cross-section
        box("helmholtz_substeps", 320, 192, 128, "DD DD PP", path="helmholtz", stretch=1.5),
        # the pressure step of a channel flow: divergence, solve, velocity update
        box("project_channel", 256, 192, 256, "PP NN PP", path="project", stretch=1.6),
        # uneven boxes with every pair of conditions, one call
        dict(name="batch_24_mixed", path="batch", count=24, size_seed=4, lo=64, hi=384, zlo=64, zhi=256,
             precision="mixed"),
        # a burst of requests of random size through the server
        dict(name="serve_32", path="serve", count=32, size_seed=5, lo=32, hi=320, zlo=32, zhi=320,
             precision="mixed", slots=8),
        # the comparison solver on a cube
        box("mg3d_box_256", 256, 256, 256, "DD NN NN", path="mg3d"),
        # the z transform alone at a length that is no power of two
        box("transform_360", 384, 256, 360, "NN NN ND", path="transform"),
        # operator, residual check and divergence at an ordinary size
        box("operator_320", 320, 256, 256, "DD NN PP", path="operator", stretch=1.2),
    ]


def draw(rng):
    """One more case: sizes spread over the logarithm of the ranges, any conditions."""
    def size(lo, hi, step=1):
        return max(lo, min(hi, step * round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)))

    path = rng.choice(["solve", "solve", "solve", "solve", "helmholtz", "project", "batch", "serve", "mg3d",
                       "transform", "operator"])
    prec = rng.choice(["fp64", "mixed"])
    if path in ("batch", "serve"):
        return dict(path=path, count=rng.randint(4, 32), size_seed=rng.randrange(1 << 30), lo=32, hi=rng.randint(96, 384),
                    zlo=32, zhi=rng.randint(64, 256), precision="mixed" if path == "serve" else prec,
                    **({"slots": rng.choice([2, 4, 8])} if path == "serve" else {}))
    if path == "solve" and rng.random() < 0.4:
        shape = rng.choice(["lshape", "obstacle"])
        return dict(path=path, shape=shape, n=size(24, 320 if shape == "lshape" else 96, rng.choice([1, 4, 16])),
                    nz=2 * size(8, 288), stretch=round(rng.uniform(0.0, 1.8), 3) if shape == "lshape" else 0.0,
                    precision=prec, retire=rng.random() < 0.8)
    most = {"mg3d": 256, "operator": 384, "transform": 384}.get(path, 512)
    step = rng.choice([1, 2, 16, 32])
    nx, ny, nz = size(32, most, step), size(32, most, step), 2 * size(16, most // 2, rng.choice([1, 8, 16]))
    pairs = " ".join(rng.choice(KINDS) for _ in range(3))
    if path == "project":
        pairs = rng.choice(["PP NN PP", "NN NN PP", "NN NN NN", "ND NN PP", "PP PP NN"])
    return dict(path=path, shape="box", nx=nx, ny=ny, nz=nz, pairs=pairs,
                stretch=rng.choice([0.0, round(rng.uniform(1.0, 2.0), 3)]), precision=prec if path == "solve" else "fp64",
                retire=rng.random() < 0.8)


# ---- problems ---------------------------------------------------------------

def faces(n, lo, hi, factor=0.0):
    """n + 1 face coordinates on [lo, hi], clustered toward both ends (tanh) when factor > 0."""
    s = np.arange(n + 1, dtype=np.float64) / n
    x = s if factor == 0.0 else 0.5 * (1.0 + np.tanh(factor * (s - 0.5)) / math.tanh(0.5 * factor))
    x[0], x[-1] = 0.0, 1.0
    return lo + (hi - lo) * x


def block(lo, nx, ny, xf, yf, bc):
    return SimpleNamespace(lo=lo, hi=(lo[0] + nx - 1, lo[1] + ny - 1), xf=xf, yf=yf, bc=bc)


def box_problem(nx, ny, nz, pairs, stretch=(0.0, 0.0)):
    px, py, pz = pairs.split()
    xf = faces(nx, 0.0, nx * H, 0.0 if px == "PP" else stretch[0])
    yf = faces(ny, 0.0, ny * H, 0.0 if py == "PP" else stretch[1])
    return SimpleNamespace(blocks=[block((1, 1), nx, ny, xf, yf, PAIRS[px] + PAIRS[py])], nz=nz, lz=nz * H,
                           zbc=PAIRS[pz], ncells=nx * ny * nz, pairs=pairs)


def lshape_problem(n, nz, factor):
    xa, xb, ya, yc = faces(n, 0.0, 1.0), faces(n, 1.0, 2.0), faces(n, 0.0, 1.0, factor), faces(n, 1.0, 2.0, factor)
    blocks = [block((1, 1), n, n, xa, ya, (N, C, N, C)), block((n + 1, 1), n, n, xb, ya, (C, N, N, N)),
              block((1, n + 1), n, n, xa, yc, (N, N, C, N))]
    return SimpleNamespace(blocks=blocks, nz=nz, lz=nz / n, zbc=(P, P), ncells=3 * n * n * nz, pairs=None)


def obstacle_problem(n, nz):
    """A 3 x 3 arrangement minus its centre: widths 2, 1, 2 and heights 1, 1, 1 of n cells a unit."""
    x0, y0, blocks = [0, 2, 3, 5], [0, 1, 2, 3], []
    for r in range(3):
        for c in range(3):
            if r == 1 and c == 1:
                continue
            nx, ny = (x0[c + 1] - x0[c]) * n, n
            bc = (N if c == 0 or (r == 1 and c == 2) else C, D if c == 2 else (N if r == 1 and c == 0 else C),
                  D if r == 0 else (N if c == 1 and r == 2 else C), D if r == 2 else (N if c == 1 and r == 0 else C))
            blocks.append(block((x0[c] * n + 1, y0[r] * n + 1), nx, ny, faces(nx, float(x0[c]), float(x0[c + 1])),
                                faces(ny, float(y0[r]), float(y0[r + 1])), bc))
    return SimpleNamespace(blocks=blocks, nz=nz, lz=nz / n, zbc=(P, P), ncells=14 * n * n * nz, pairs=None)


def problem_of(case):
    if case["shape"] == "lshape":
        return lshape_problem(case["n"], case["nz"], case["stretch"])
    if case["shape"] == "obstacle":
        return obstacle_problem(case["n"], case["nz"])
    return box_problem(case["nx"], case["ny"], case["nz"], case["pairs"], (case["stretch"], case["stretch"]))


def problems_of(case):
    """The boxes of a batch or a burst: sizes of multiples of 16, every pair of conditions."""
    rng = random.Random(case["size_seed"])
    out = []
    for _ in range(case["count"]):
        s = lambda lo, hi: min(hi // 16 * 16, max(lo, 16 * round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 16)))  # noqa: E731
        nx, ny, nz = s(case["lo"], case["hi"]), s(case["lo"], case["hi"]), s(case["zlo"], case["zhi"])
        pairs = " ".join(rng.choice(KINDS) for _ in range(3))
        f = (0.0, 0.0) if case["path"] == "batch" else (rng.uniform(1.0, 2.0), rng.uniform(1.0, 2.0))
        out.append(box_problem(nx, ny, nz, pairs, f))
    return out


ALPHAS = (40.0, 90.0, 160.0)  # alpha h^2 between 2e-3 and 1e-2: a few time steps per cell diffusion time


# ---- inputs -------------------------------------------------------------------

def field(n, gen):
    return torch.rand(n, generator=gen, device="cuda", dtype=torch.float64).mul_(2.0).sub_(1.0)


def velocity(prob, gen):
    """A random predicted velocity: faces on a periodic seam equal, wall-normal components zero at Neumann walls."""
    b = prob.blocks[0]
    nz, ny, nx = prob.nz, b.hi[1], b.hi[0]
    u = field(nz * ny * (nx + 1), gen).view(nz, ny, nx + 1)
    v = field(nz * (ny + 1) * nx, gen).view(nz, ny + 1, nx)
    nzw = nz if prob.zbc[0] == P else nz + 1
    w = field(nzw * ny * nx, gen).view(nzw, ny, nx)
    for t, dim, lo, hi in ((u, 2, b.bc[0], b.bc[1]), (v, 1, b.bc[2], b.bc[3]), (w, 0, prob.zbc[0], prob.zbc[1])):
        n = t.shape[dim] - 1
        if lo == P:
            if dim:
                t.select(dim, n).copy_(t.select(dim, 0))
            continue
        if lo == N:
            t.select(dim, 0).zero_()
        if hi == N:
            t.select(dim, n).zero_()
    return u.reshape(-1), v.reshape(-1), w.reshape(-1)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    path = case["path"]
    s = SimpleNamespace(case=case, path=path)
    if path in ("batch", "serve"):
        s.probs = problems_of(case)
        s.rhs = [field(p.ncells, gen) for p in s.probs]
        s.p = [torch.zeros(p.ncells, device="cuda", dtype=torch.float64) for p in s.probs]
        if path == "batch":
            s.plans = [mbp.Plan(p, precision=case["precision"]) for p in s.probs]
        else:
            s.server = mbp.Server(8 << 30, slots=case["slots"], precision=case["precision"])
        return s
    s.prob = problem_of(case)
    n = s.prob.ncells
    if path == "mg3d":
        s.plan = mbp.Plan3D(s.prob)
    else:
        s.plan = mbp.Plan(s.prob, precision=case["precision"])
    s.flags = mbp.PROJECT_RHS | (mbp.RETIRE if case["retire"] else 0)
    if path == "helmholtz":
        s.rhs = [field(n, gen) for _ in ALPHAS]
        s.p = [torch.zeros(n, device="cuda", dtype=torch.float64) for _ in ALPHAS]
    elif path == "project":
        s.star = velocity(s.prob, gen)
        s.vel = tuple(torch.empty_like(t) for t in s.star)
        s.phi, s.tmp = (torch.zeros(n, device="cuda", dtype=torch.float64) for _ in range(2))
    elif path == "operator":
        s.rhs, s.x = field(n, gen), field(n, gen)
        s.vel = velocity(s.prob, gen)
        s.p, s.div = (torch.zeros(n, device="cuda", dtype=torch.float64) for _ in range(2))
    else:
        s.rhs = field(n, gen)
        s.p = torch.zeros(n, device="cuda", dtype=torch.float64)
        if path == "transform":
            s.hat = torch.zeros(n, device="cuda", dtype=torch.float64)
    return s


def run(s):
    if s.path == "solve":
        s.plan.solve(s.rhs, s.p, rtol=RTOL, flags=s.flags)
        return s.p
    if s.path == "helmholtz":
        for a, f, p in zip(ALPHAS, s.rhs, s.p):
            s.plan.set_helmholtz(a)
            s.plan.solve(f, p, rtol=RTOL, flags=s.flags)
        return s.p
    if s.path == "project":
        for t, f in zip(s.vel, s.star):  # this step's predicted velocity
            t.copy_(f)
        s.plan.project(*s.vel, GAMMA_DT, s.phi, s.tmp, rtol=RTOL, flags=s.flags)
        return [*s.vel, s.phi]
    if s.path == "batch":
        mbp.solve_batch(s.plans, s.rhs, s.p, rtol=RTOL, flags=mbp.PROJECT_RHS)
        return s.p
    if s.path == "serve":
        tickets = [s.server.submit(pr, f, p, rtol=RTOL, flags=mbp.PROJECT_RHS) for pr, f, p in zip(s.probs, s.rhs, s.p)]
        for t in tickets:
            status = s.server.wait(t)[0]
            if status != mbp.OK:
                raise mbp.MBPError(status, "serve")
        return s.p
    if s.path == "mg3d":
        s.plan.solve(s.rhs, s.p, rtol=RTOL, flags=mbp.PROJECT_RHS)
        return s.p
    if s.path == "transform":
        s.plan.forward(s.rhs, s.hat)
        s.plan.inverse(s.hat, s.p)
        return s.hat, s.p
    s.plan.apply(s.x, s.p)
    norm = s.plan.residual_norm(s.rhs, s.x)
    s.plan.divergence(*s.vel, s.div, scale=1.0 / GAMMA_DT)
    return s.p, norm, s.div


GAMMA_DT = 0.01


def work(case):
    """Bytes: inputs read once, outputs written once.  Operations of a solve: both transforms
    (2.5 n log2 n per column) and six V-cycles of red-black sweeps, residual and transfers on a
    hierarchy of 4/3 of the plane (about 40 per cell and cycle)."""
    def solve_flops(cells, nz):
        return cells * (5.0 * math.log2(nz) + 6 * 40 * 4.0 / 3.0)

    path = case["path"]
    if path in ("batch", "serve"):
        ps = problems_of(case)
        return {"bytes": sum(16.0 * p.ncells for p in ps), "flops": sum(solve_flops(p.ncells, p.nz) for p in ps)}
    p = problem_of(case)
    n = float(p.ncells)
    if path == "transform":
        return {"bytes": 32 * n, "flops": 5.0 * n * math.log2(p.nz)}
    if path == "operator":
        return {"bytes": (16 + 16 + 32) * n, "flops": 40 * n}
    if path == "project":
        return {"bytes": 56 * n, "flops": solve_flops(n, p.nz) + 20 * n}
    if path == "mg3d":
        return {"bytes": 16 * n, "flops": 10 * 80 * 8.0 / 7.0 * n}
    k = len(ALPHAS) if path == "helmholtz" else 1
    return {"bytes": 16 * n * k, "flops": k * solve_flops(n, p.nz)}


# ---- dense 64-bit references (boxes) ---------------------------------------------

def line(xf, lo, hi):
    """1D finite-volume second difference diag(1/dc) K on faces xf: (K, dc) with K symmetric."""
    xf = torch.as_tensor(xf, dtype=torch.float64, device="cuda")
    dc = xf[1:] - xf[:-1]
    n = dc.numel()
    K = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    w = 2.0 / (dc[1:] + dc[:-1])
    i = torch.arange(n - 1, device="cuda")
    K[i, i + 1] += w
    K[i + 1, i] += w
    if lo == P:
        s = 2.0 / (dc[0] + dc[-1])
        K[0, n - 1] += s
        K[n - 1, 0] += s
    K -= torch.diag(K.sum(1))
    if lo == D:
        K[0, 0] -= 2.0 / dc[0]
    if hi == D:
        K[n - 1, n - 1] -= 2.0 / dc[-1]
    return K, dc


def axes_of(prob):
    b = prob.blocks[0]
    zf = np.arange(prob.nz + 1) * (prob.lz / prob.nz)
    return [line(zf, *prob.zbc), line(b.yf, b.bc[2], b.bc[3]), line(b.xf, b.bc[0], b.bc[1])]


def along(M, t, dim):
    """Matrix M applied along dimension dim of a 3D field."""
    if dim == 2:
        return t @ M.T
    if dim == 1:
        return torch.matmul(M, t)
    return (M @ t.reshape(t.shape[0], -1)).reshape(M.shape[0], t.shape[1], t.shape[2])


def direct_solve(prob, f, alpha=0.0):
    """(L_h - alpha) p = f by eigen-decomposition of the three 1D operators; a null mode is dropped."""
    ax = axes_of(prob)
    lam, V, sw = [], [], []
    for K, dc in ax:
        r = dc.sqrt()
        e, v = torch.linalg.eigh(K / r[:, None] / r[None, :])
        lam.append(e)
        V.append(v)
        sw.append(r)
    t = f.view(*(a[1].numel() for a in ax)) * sw[0][:, None, None] * sw[1][:, None] * sw[2]
    for d in range(3):
        t = along(V[d].T.contiguous(), t, d)
    mu = lam[0][:, None, None] + lam[1][:, None] + lam[2] - alpha
    top = max(float(e.abs().max()) for e in lam)
    t = torch.where(mu.abs() > 1e-11 * top, t / mu, torch.zeros_like(t))
    del mu
    for d in range(3):
        t = along(V[d], t, d)
    return (t / sw[0][:, None, None] / sw[1][:, None] / sw[2]).reshape(-1)


def basis(kind, n):
    """Orthonormal eigenvectors of the uniform line as columns, in the library's modal order."""
    j = torch.arange(n, dtype=torch.float64, device="cuda")[:, None]
    q = torch.arange(n, dtype=torch.float64, device="cuda")[None, :]
    c = math.sqrt(2.0 / n)
    if kind == "PP":
        th = 2.0 * math.pi * ((q * j) % n) / n
        return (torch.cos(th) + torch.sin(th)) / math.sqrt(n)
    if kind == "NN":
        T = torch.cos(math.pi * ((q * (2 * j + 1)) % (4 * n)) / (2 * n)) * c
        T[:, 0] = 1.0 / math.sqrt(n)
        return T
    if kind == "DD":
        T = torch.sin(math.pi * (((q + 1) * (2 * j + 1)) % (4 * n)) / (2 * n)) * c
        T[:, n - 1] /= math.sqrt(2.0)
        return T
    th = math.pi * (((2 * q + 1) * (2 * j + 1)) % (8 * n)) / (4 * n)
    return (torch.cos(th) if kind == "ND" else torch.sin(th)) * c


def diverge(prob, u, v, w, scale):
    (_, dz), (_, dy), (_, dx) = axes_of(prob)
    nz, ny, nx = prob.nz, dy.numel(), dx.numel()
    u, v = u.view(nz, ny, nx + 1), v.view(nz, ny + 1, nx)
    w = w.view(-1, ny, nx)
    if w.shape[0] == nz:
        w = torch.cat([w, w[:1]])
    return scale * ((u[:, :, 1:] - u[:, :, :-1]) / dx + (v[:, 1:] - v[:, :-1]) / dy[:, None]
                    + (w[1:] - w[:-1]) / dz[:, None, None])


def gradient(prob, phi, dim, periodic_faces):
    """Face gradient of a cell field along one dimension."""
    dc = axes_of(prob)[dim][1]
    lo, hi = [prob.zbc, prob.blocks[0].bc[2:4], prob.blocks[0].bc[0:2]][dim]
    t = phi.movedim(dim, -1)
    left, right = (t[..., -1:], t[..., :1]) if lo == P else (-t[..., :1] if lo == D else t[..., :1],
                                                              -t[..., -1:] if hi == D else t[..., -1:])
    t = torch.cat([left, t, right], -1)
    dl, dr = (dc[-1:], dc[:1]) if lo == P else (dc[:1], dc[-1:])
    g = (t[..., 1:] - t[..., :-1]) / (0.5 * (torch.cat([dl, dc]) + torch.cat([dc, dr])))
    if lo == P and not periodic_faces:
        g = g[..., :-1]
    return g.movedim(-1, dim)


def exact(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    path = case["path"]
    if path in ("batch", "serve"):
        probs = problems_of(case)
        rhs = [field(p.ncells, gen) for p in probs]
        return [direct_solve(p, f) for p, f in zip(probs, rhs)]
    if case["shape"] != "box":
        return None  # no separable form; a sparse solve of every mode takes minutes
    prob = problem_of(case)
    n = prob.ncells
    if path == "helmholtz":
        rhs = [field(n, gen) for _ in ALPHAS]
        return [direct_solve(prob, f, a) for a, f in zip(ALPHAS, rhs)]
    if path == "project":
        u, v, w = velocity(prob, gen)
        phi = direct_solve(prob, diverge(prob, u, v, w, 1.0 / GAMMA_DT).reshape(-1))
        f = phi.view(prob.nz, prob.blocks[0].hi[1], prob.blocks[0].hi[0])
        for t, dim in ((u, 2), (v, 1), (w, 0)):
            t.sub_(GAMMA_DT * gradient(prob, f, dim, dim > 0).reshape(-1))
        return [u, v, w, phi]
    if path == "operator":
        rhs, x = field(n, gen), field(n, gen)
        u, v, w = velocity(prob, gen)
        ax = axes_of(prob)
        t = x.view(*(a[1].numel() for a in ax))
        Lx = sum(along(K / dc[:, None], t, d) for d, (K, dc) in enumerate(ax)).reshape(-1)
        norm = torch.stack([(rhs - Lx).norm(), rhs.norm()])
        return Lx, norm, diverge(prob, u, v, w, 1.0 / GAMMA_DT).reshape(-1)
    rhs = field(n, gen)
    if path == "transform":
        hat = basis(prob.pairs.split()[2], prob.nz).T @ rhs.view(prob.nz, -1)
        return hat.reshape(-1), rhs
    return direct_solve(prob, rhs)
