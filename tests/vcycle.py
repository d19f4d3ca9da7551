"""One multigrid V-cycle of every mode, written out in float64 numpy (test infrastructure).

The cycle the library documents: one red-black Gauss-Seidel sweep, area-weighted
restriction of the residual, the next level's cycle from zero, bilinear correction with
physical weights, one more sweep; an exact solve (null mode dropped) on the coarsest
plane.  It shares no code with the library; operators and transforms are the oracle's.
Every kernel that runs part of a cycle must leave this iterate, cell by cell, so a
wrong transfer or a stale cell cannot hide behind convergence.
"""
import copy

import numpy as np
import scipy.sparse as sp

import oracle
from oracle.grid import DIRICHLET, PERIODIC, XM, XP, YM, YP


def _merge(f):
    """Faces of the next level: pairs of cells, an odd count's last three."""
    n = len(f) - 1
    return np.array([f[2 * i] for i in range(n // 2)] + [f[n]])


def _level(g, bx, by):
    c = copy.copy(g)
    c.xf = [_merge(f) if bx else f for f in g.xf]
    c.yf = [_merge(f) if by else f for f in g.yf]
    c.nx, c.ny = [len(f) - 1 for f in c.xf], [len(f) - 1 for f in c.yf]
    c.dcx, c.dcy = [np.diff(f) for f in c.xf], [np.diff(f) for f in c.yf]
    c.xc, c.yc = [0.5 * (f[1:] + f[:-1]) for f in c.xf], [0.5 * (f[1:] + f[:-1]) for f in c.yf]
    c.off2 = list(np.concatenate([[0], np.cumsum([a * b for a, b in zip(c.nx, c.ny)])]).astype(int))
    c.ncell2 = c.off2[-1]
    return c


def hierarchy(prob):
    """Geometries of every level: each step halves the direction of the smaller mean width,
    or both within a factor of sqrt(2), while every block has four cells along it."""
    levels = [oracle.Geometry(prob)]
    while True:
        g = levels[-1]
        hx = sum(f[-1] - f[0] for f in g.xf) / sum(g.nx)
        hy = sum(f[-1] - f[0] for f in g.yf) / sum(g.ny)
        bx, by = not hy < np.sqrt(0.5) * hx, not hx < np.sqrt(0.5) * hy
        if (bx and min(g.nx) < 4) or (by and min(g.ny) < 4):
            break
        levels.append(_level(g, bx, by))
    assert levels[-1].ncell2 <= 256, "coarsens per class of blocks, which is not written out here"
    return levels


def colours(g):
    """Cell indices by colour: joined neighbours differ; a ring of odd length takes two more."""
    par = [-1] * g.nb
    for s in range(g.nb):
        if par[s] >= 0:
            continue
        par[s], stack = 0, [s]
        while stack:
            b = stack.pop()
            for f in range(4):
                k = g.nbr[b][f]
                if k < 0 or par[k] >= 0:
                    continue
                n = g.nx[b] if f == XP else g.nx[k] if f == XM else g.ny[b] if f == YP else g.ny[k]
                par[k] = (par[b] + n) & 1
                stack.append(k)
    col = np.empty(g.ncell2, dtype=int)
    for b in range(g.nb):
        j, i = np.meshgrid(np.arange(g.ny[b]), np.arange(g.nx[b]), indexing="ij")
        c = (i + j + par[b]) & 1
        kx, ky = g.nbr[b][XP], g.nbr[b][YP]
        odd = np.zeros_like(c, dtype=bool)
        if kx >= 0 and (par[b] + g.nx[b] + par[kx]) & 1:
            odd |= i == g.nx[b] - 1
        if ky >= 0 and (par[b] + g.ny[b] + par[ky]) & 1:
            odd |= j == g.ny[b] - 1
        col[g.off2[b]:g.off2[b + 1]] = (c + 2 * odd).ravel()
    return [np.nonzero(col == c)[0] for c in range(4) if (col == c).any()]


def _axis(F, G, below, above):
    """Per fine cell of one block along one axis: parent, restriction weight, lower coarse
    neighbour and its weight.  below / above: widths beyond the ends (None: a wall)."""
    n, nc = len(F) - 1, len(G) - 1
    ratio = 1 if n == nc else 2
    parent = np.minimum(np.arange(n) // ratio, nc - 1)
    rw = np.diff(F) / np.diff(G)[parent]
    c = 0.5 * (G[1:] + G[:-1])
    lo = 2 * G[0] - c[0] if below is None else G[0] - 0.5 * below
    hi = 2 * G[-1] - c[-1] if above is None else G[-1] + 0.5 * above
    ext = np.concatenate([[lo], c, [hi]])
    x = 0.5 * (F[1:] + F[:-1])
    t = np.minimum(np.searchsorted(ext[1:], x, side="right"), nc)
    return parent, rw, t - 1, (ext[t + 1] - x) / (ext[t + 1] - ext[t])


def transfers(g, c):
    """Sparse restriction (fine -> coarse) and prolongation (coarse -> fine)."""
    rr, rc, rv, pr, pc, pv = [], [], [], [], [], []
    for b in range(g.nb):
        def beyond(f, d):
            k = g.nbr[b][f]
            return None if k < 0 else d[k][-1 if f in (XM, YM) else 0]
        ax = _axis(g.xf[b], c.xf[b], beyond(XM, c.dcx), beyond(XP, c.dcx))
        ay = _axis(g.yf[b], c.yf[b], beyond(YM, c.dcy), beyond(YP, c.dcy))
        for j in range(g.ny[b]):
            for i in range(g.nx[b]):
                me = g.off2[b] + j * g.nx[b] + i
                rr.append(c.off2[b] + ay[0][j] * c.nx[b] + ax[0][i])
                rc.append(me)
                rv.append(ax[1][i] * ay[1][j])
                for dj in (0, 1):
                    for di in (0, 1):
                        k, s, I, J = b, 1.0, ax[2][i] + di, ay[2][j] + dj
                        # one cell beyond a face: the partner's (y first), or a wall's mirror image
                        if J < 0 or J >= c.ny[k]:
                            f = YM if J < 0 else YP
                            if g.nbr[k][f] >= 0:
                                k = g.nbr[k][f]
                                J = c.ny[k] - 1 if f == YM else 0
                            else:
                                s *= -1.0 if g.bc[k][f] == DIRICHLET else 1.0
                                J = 0 if f == YM else c.ny[k] - 1
                        if I < 0 or I >= c.nx[k]:
                            f = XM if I < 0 else XP
                            if g.nbr[k][f] >= 0:
                                k = g.nbr[k][f]
                                I = c.nx[k] - 1 if f == XM else 0
                            else:
                                s *= -1.0 if g.bc[k][f] == DIRICHLET else 1.0
                                I = 0 if f == XM else c.nx[k] - 1
                        pr.append(me)
                        pc.append(c.off2[k] + J * c.nx[k] + I)
                        pv.append(s * (ax[3][i] if di == 0 else 1 - ax[3][i]) * (ay[3][j] if dj == 0 else 1 - ay[3][j]))
    return (sp.csr_matrix((rv, (rr, rc)), shape=(c.ncell2, g.ncell2)),
            sp.csr_matrix((pv, (pr, pc)), shape=(g.ncell2, c.ncell2)))


class Cycle:
    """The cycles of one problem; fields are (modes, plane) in the packed plane order."""

    def __init__(self, prob, alpha=0.0):
        self.prob, self.g = prob, hierarchy(prob)
        self.T = oracle.basis(self.g[0].zkind, self.g[0].nz)
        lam = oracle.eigenvalues(self.g[0].zkind, self.g[0].nz)
        self.sig = (lam / self.g[0].dz ** 2 - alpha)[:, None]
        self.A = [oracle.assemble_2d(g).tocsr() for g in self.g]
        self.d = [a.diagonal() for a in self.A]
        self.col = [colours(g) for g in self.g]
        self.rows = [[a[c] for c in col] for a, col in zip(self.A, self.col)]
        self.move = [transfers(g, c) for g, c in zip(self.g, self.g[1:])]
        area = self.g[-1].areas()
        r = np.sqrt(area)
        S = self.A[-1].toarray() * r[:, None] / r[None, :]
        self.mu, V = np.linalg.eigh(0.5 * (S + S.T))
        self.wl, self.wr = V / r[:, None], V.T * r[None, :]

    def modes(self, f):
        g = self.g[0]
        return np.concatenate([self.T.T @ b.reshape(g.nz, -1) for b in g.split3(np.asarray(f))], axis=1)

    def field(self, x):
        g = self.g[0]
        return np.concatenate([(self.T @ x[:, g.off2[b]:g.off2[b + 1]]).ravel() for b in range(g.nb)])

    def apply(self, l, x):
        return (self.A[l] @ x.T).T + self.sig * x

    def sweep(self, l, x, f):
        for c, rows in zip(self.col[l], self.rows[l]):
            d = self.d[l][c] + self.sig
            x[:, c] = (f[:, c] - (rows @ x.T).T + self.d[l][c] * x[:, c]) / d

    def cycle(self, x, f, l=0):
        if l + 1 == len(self.g):
            den = self.mu[None, :] + self.sig
            top = np.abs(self.mu).max() + np.abs(self.sig)
            b = f @ self.wr.T
            return np.where(np.abs(den) > 1e-11 * top, b / np.where(den == 0, 1.0, den), 0.0) @ self.wl.T
        self.sweep(l, x, f)
        R, P = self.move[l]
        fc = (R @ (f - self.apply(l, x)).T).T
        x += (P @ self.cycle(np.zeros_like(fc), fc, l + 1).T).T
        self.sweep(l, x, f)
        return x

    def solve(self, f, cycles, inner=1, start=None):
        """The field after so many cycles (inner > 1: refinement steps of that many each)."""
        g = self.g[0]
        fh = self.modes(f)
        sing = oracle.is_singular(self.prob)
        area = g.areas()
        if sing:
            fh[0] -= area @ fh[0] / area.sum()
        x = np.zeros_like(fh) if start is None else self.modes(start)
        for _ in range(cycles):
            r = fh - self.apply(0, x)
            e = np.zeros_like(x)
            for _ in range(inner):
                e = self.cycle(e, r)
            x = x + e
        if sing:
            x[0] -= area @ x[0] / area.sum()
        return self.field(x)


def tolerance(prob, bits, cycles):
    """Largest cell difference against the largest value that rounding explains: eight
    roundings a residual, amplified by at most the square of the cells across the plane."""
    n = max(sum(b.nx for b in prob.blocks), sum(b.ny for b in prob.blocks))
    return 8.0 * 2.0 ** -bits * n * n * cycles
