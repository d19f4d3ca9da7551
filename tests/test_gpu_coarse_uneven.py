"""Joined blocks whose colours are uneven on a level that would run in LDS: a T of even
blocks with 4096 cells (513 and 511 cells of the two colours on its second level), the
same at twice the size, and a grid of odd blocks.

After each of the first cycles the error is at most a tenth above the one of the cycle
written out in numpy (whose interpolation beside a re-entrant corner may differ), and the
converged field meets the solver's bounds in every cell: 10 rtol of the largest value times
the square root of the cells (an L2 bound seen by one cell) is far above what is asked."""
import numpy as np
import pytest

import oracle
import vcycle
import workloads as W
from test_gpu_pair import C, D, N, _grid

pytestmark = pytest.mark.gpu


def _tee(s, nz=4):
    h = 1.0 / (64.0 * s)
    spec = [((34, 30), (30, 34), (C, C, C, D)), ((0, 30), (34, 34), (D, C, N, N)), ((64, 30), (30, 34), (C, N, D, N)),
            ((34, 0), (30, 30), (N, D, N, C))]
    blocks = []
    for (x, y), (nx, ny), bc in spec:
        x, y, nx, ny = x * s, y * s, nx * s, ny * s
        blocks.append(W.Block((x + 1, y + 1), (x + nx, y + ny), W.faces(nx, x * h, (x + nx) * h),
                              W.faces(ny, y * h, (y + ny) * h), bc))
    return W.Problem(blocks=blocks, nz=nz, lz=nz * h, zbc=W.PAIRS["NN"], name=f"tee{s}")


PROBLEMS = [_tee(1), _tee(2), _grid([9] * 5, [9] * 5, [], [D, N])]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("prob", PROBLEMS, ids=lambda p: p.name)
def test_uneven_colours(prob, precision):
    import torch
    import paper_2106_03583_amd as m
    print(f"uneven colours {prob.name} {precision}", flush=True)
    f = W.rhs(prob, 61)
    want, ref = oracle.solve(prob, f), vcycle.Cycle(prob)
    fd = torch.from_numpy(f).cuda()
    for cycles in (1, 2, 3, 4):
        plan = m.Plan(prob, precision=precision, max_cycles=cycles, inner=1)
        p = torch.zeros_like(fd)
        plan.solve(fd, p, rtol=1e-15, flags=m.RETIRE, raise_on_error=False)
        plan.close()
        got, exp = oracle.rel_error(p.cpu().numpy(), want), oracle.rel_error(ref.solve(f, cycles), want)
        assert got <= 1.1 * exp, (cycles, got, exp)
    plan = m.Plan(prob, precision=precision)
    p = torch.zeros_like(fd)
    plan.solve(fd, p, rtol=1e-10, flags=m.RETIRE)
    got = p.cpu().numpy()
    assert oracle.rel_residual(prob, got, f) <= 1e-10
    assert oracle.rel_error(got, want) <= 1e-9
    assert np.abs(got - want).max() <= 1e-9 * np.abs(want).max() * np.sqrt(prob.ncells)
    plan.close()
