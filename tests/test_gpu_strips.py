"""Levels the pair march does not take, now that it takes odd sides at walls: odd sides at
joined faces (strip kernels, one or two levels of them), an odd ring (the plain sweeps), and
an odd ring below a level of the march.  Single cycles cell by cell, alone and in a group
beside marched problems (whose FP32 correction is added by the march, theirs by a pass of
its own); both pre-smoothing forms and two sweeps against the oracle (the register march
smooths the cells along an odd joined face in another order, so its single cycles differ).

Tolerances: single cycles as in test_gpu_cycle_cells.py, solves 1e-10 on the residual and
1e-9 on the error."""
import numpy as np
import pytest

import oracle
import vcycle
import workloads as W
from test_gpu_pair import D, N, _box, _grid

pytestmark = pytest.mark.gpu

STRIPS = [_grid([75, 83], [60, 91], [], [D, N]), _grid([91, 120, 75], [60, 65], [], [N, D]), _grid([57, 60], [40, 64], [], [D, N])]
OTHERS = [_box(75, 82, "PP", "DD"), W.box(302, 256, 4, 302 / 128, 2.0, 4 / 128, "PP", "NN", "DD", name="ring302")]
MARCHED = [_box(112, 90, "DD", "NN"), _box(113, 92, "DD", "NN")]


def _cells(prob, got, want, bits, n):
    across = max(sum(b.nx for b in prob.blocks), sum(b.ny for b in prob.blocks))
    off = np.abs(got - want).max() / np.abs(want).max()
    assert off <= 8.0 * 2.0 ** -bits * across * n, (prob.name, off)


@pytest.mark.parametrize("prob", STRIPS + OTHERS[:1], ids=lambda p: p.name)
def test_cells_of_strip_cycles(prob):
    import torch
    import paper_2106_03583_amd as m
    print(f"strips {prob.name}", flush=True)
    ref = vcycle.Cycle(prob)
    f = W.rhs(prob, 21)
    fd = torch.from_numpy(f).cuda()
    for cycles in (1, 2):
        for precision, bits, inner in (("fp64", 53, 1), ("mixed", 24, 1), ("mixed", 24, 2)):
            plan = m.Plan(prob, precision=precision, max_cycles=cycles, inner=inner)
            p = torch.zeros_like(fd)
            plan.solve(fd, p, rtol=1e-15, flags=m.PROJECT_RHS | m.RETIRE, raise_on_error=False)
            _cells(prob, p.cpu().numpy(), ref.solve(f, cycles, inner), bits, inner * cycles)
            plan.close()


@pytest.mark.parametrize("inner", [1, 2, 3])
def test_cells_of_a_group_with_strips(inner):
    import torch
    import paper_2106_03583_amd as m
    probs = STRIPS + MARCHED
    f = [W.rhs(p, 22 + i) for i, p in enumerate(probs)]
    fd = [torch.from_numpy(a).cuda() for a in f]
    plans = [m.Plan(p, precision="mixed", max_cycles=2, inner=inner) for p in probs]
    for flags in (m.AUTOTUNE, 0):
        x = [torch.zeros_like(a) for a in fd]
        m.solve_batch(plans, fd, x, rtol=1e-15, flags=m.PROJECT_RHS | flags, raise_on_error=False)
        assert m.batch_schedule(plans)[0] == 0  # all grouped
        for p, a, b in zip(probs, f, x):
            _cells(p, b.cpu().numpy(), vcycle.Cycle(p).solve(a, 2, inner), 24, 2 * inner)
    for pl in plans:
        pl.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("prob", STRIPS + OTHERS + MARCHED, ids=lambda p: p.name)
def test_forms_and_sweeps(prob, precision):
    import torch
    import paper_2106_03583_amd as m
    f = W.rhs(prob, 23)
    want = oracle.solve(prob, f)
    fp = oracle.project_compatible(prob, f) if oracle.is_singular(prob) else f
    fd = torch.from_numpy(f).cuda()
    for kw in ({"march": 1}, {"march": 1, "nu1": 2, "nu2": 2}, {"nu1": 2, "nu2": 2}, {"nu1": 2, "nu2": 1}):
        plan = m.Plan(prob, precision=precision, **kw)
        for flags in (0, m.RETIRE):
            p = torch.zeros_like(fd)
            plan.solve(fd, p, rtol=1e-10, flags=m.PROJECT_RHS | flags)
            got = p.cpu().numpy()
            assert oracle.rel_residual(prob, got, fp) <= 1e-10
            assert oracle.rel_error(got, want) <= 1e-9
        plan.close()
