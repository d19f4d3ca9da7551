"""The pair march at the sizes where it can go wrong: strip widths around its
112 / 120 column limits, strips that end inside the ring of 16 rows, the
smallest blocks it takes, rings, walls of every kind, joined blocks whose
vertical neighbours differ; and planes just outside its rule.

Tolerances: the stopping rule bounds the 3D residual by rtol and the relative
error by etol = 10 rtol (both 1e-10 / 1e-9 here), in every precision."""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import oracle  # noqa: E402
import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu
D, N, C = W.DIRICHLET, W.NEUMANN, W.CONNECT


def _box(nx, ny, xp, yp, zp="PP", nz=6, fx=0.0, fy=0.0):
    return W.box(nx, ny, nz, nx / 64.0, ny / 64.0, nz / 64.0, xp, yp, zp, xfactor=fx, yfactor=fy,
                 name=f"{nx}x{ny}_{xp}{yp}{zp}")


def _grid(widths, heights, missing, walls, nz=4):
    """Blocks of a column / row grid, some missing, outer faces from `walls` in turn."""
    h = 1.0 / 64.0
    x0, y0 = np.concatenate([[0], np.cumsum(widths)]), np.concatenate([[0], np.cumsum(heights)])
    have = {(i, j) for i in range(len(widths)) for j in range(len(heights))} - set(missing)
    blocks, k = [], 0
    for j, ny in enumerate(heights):
        for i, nx in enumerate(widths):
            if (i, j) not in have:
                continue
            bc = []
            for d in ((-1, 0), (1, 0), (0, -1), (0, 1)):
                joined = (i + d[0], j + d[1]) in have
                bc.append(C if joined else walls[k % len(walls)])
                k += not joined
            lo = (int(x0[i]) + 1, int(y0[j]) + 1)
            blocks.append(W.Block(lo, (lo[0] + nx - 1, lo[1] + ny - 1), W.faces(nx, x0[i] * h, x0[i + 1] * h, 0, 0.6),
                                  W.faces(ny, y0[j] * h, y0[j + 1] * h, 0, 0.4), tuple(bc)))
    return W.Problem(blocks=blocks, nz=nz, lz=nz * h, zbc=W.PAIRS["NN"],
                     name=f"grid{widths}x{heights}-{missing}".replace(" ", ""))


PROBLEMS = [
    _box(112, 90, "DD", "NN"), _box(114, 92, "NN", "DD", "DD"), _box(226, 48, "PP", "ND", "ND"),
    _box(120, 130, "DN", "PP", "NN", fx=1.2), _box(242, 64, "PP", "PP", "PP"), _box(130, 66, "NN", "NN", "DN"),
    _box(1120, 8, "DD", "NN"), _box(8, 1100, "NN", "DD"), _box(64, 258, "ND", "DN", "PP", fy=1.5),
    _box(128, 128, "PP", "NN", "NN"), _box(113, 96, "DD", "NN"), _box(112, 91, "PP", "DD"),
    _grid([56, 60], [40, 64], [(1, 1)], [N, D]), _grid([60, 8, 56], [36, 48], [(1, 0)], [D, N, N]),
    _grid([40, 44], [8, 52, 48], [(1, 1)], [N]), _grid([64, 58], [44, 44], [], [D, N]),
    _grid([16, 120, 16], [24, 30, 24], [(1, 1)], [N, N, D]),
]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


@pytest.fixture(scope="module")
def mbp():
    import paper_2106_03583_amd as m
    return m


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("prob", PROBLEMS, ids=lambda p: p.name)
def test_pair_march(torch_cuda, mbp, prob, precision):
    torch = torch_cuda
    print(f"pair march {prob.name} {precision}", flush=True)
    f = W.rhs(prob, 41)
    ref = oracle.solve(prob, f)
    fproj = oracle.project_compatible(prob, f) if oracle.is_singular(prob) else f
    plan = mbp.Plan(prob, precision=precision)
    fd = torch.from_numpy(f).cuda()
    for flags in (0, mbp.RETIRE, mbp.RETIRE | mbp.WARM_START):
        # (the warm start begins from the converged solution scaled by a half)
        p = torch.from_numpy(0.5 * ref).cuda() if flags & mbp.WARM_START else torch.zeros_like(fd)
        plan.solve(fd, p, rtol=1e-10, flags=mbp.PROJECT_RHS | flags)
        got = p.cpu().numpy()
        assert oracle.rel_residual(prob, got, fproj) <= 1e-10
        assert oracle.rel_error(got, ref) <= 1e-9
