"""Single V-cycles of every kernel that runs part of one, cell by cell against the cycle
written out in numpy (vcycle.py): the march's forms (pre-smoothing and restriction from
zero and from an iterate, correction and post-smoothing, whole cycles, the FP32 sweep that
adds to the FP64 iterate) on even and odd planes, FP64 and FP32, alone and in grouped
launches, strips of every width and height, and the LDS-resident levels, odd rings among
them.  A wrong transfer that only slows convergence cannot pass, nor a cell that was left
from another solve on the same plan.

Tolerance: eight roundings a residual; their errors are independent from cell to cell, so
the smooth part that a cycle amplifies (by the square of the cells across) is smaller by
the number of cells across.  Interpolation beside a re-entrant corner is free to take
either neighbour's weights (2e-5 of the largest value on the layouts here); there 1e-3."""
import numpy as np
import pytest

import vcycle
import workloads as W
from test_gpu_coarse import _ring
from test_gpu_pair import D, N, _box, _grid

pytestmark = pytest.mark.gpu

EVEN = [_box(112, 90, "DD", "NN"), _box(226, 48, "PP", "ND", "ND"), _box(242, 64, "PP", "PP", "PP"),
        _box(130, 66, "NN", "NN", "DN"), _box(64, 258, "ND", "DN", "PP", fy=1.5), _box(120, 400, "DN", "PP", "NN", fx=1.2),
        _grid([64, 58], [44, 44], [], [D, N])]
ODD = [_box(113, 96, "DD", "NN"), _box(112, 91, "ND", "DD"), _box(111, 97, "NN", "DN", "NN"),
       _box(121, 65, "ND", "DD", "DN", fx=-1.2, fy=1.5), _box(225, 49, "DD", "NN", "DD", fy=-1.5),
       _box(241, 131, "NN", "DD", fx=0.7), _box(67, 259, "DD", "NN", "PP", fx=1.8, fy=1.8),
       _grid([57, 60], [40, 64], [], [D, N]), _box(75, 82, "PP", "DD")]
LDS = [_box(64, 64, "DD", "NN"), _box(65, 62, "NN", "DD"), _box(33, 31, "DD", "DN", "ND", fx=1.5),
       _box(46, 45, "NN", "NN", "DN"), _box(35, 37, "PP", "PP", "DD"), _box(32, 32, "PP", "PP", "NN"),
       _ring([24, 21, 16], 12), _grid([30, 34], [22, 20], [], [N, D])]
CORNER = [_grid([56, 60], [40, 64], [(1, 1)], [N, D]), _grid([16, 120, 16], [24, 30, 24], [(1, 1)], [N, N, D]),
          W.lshape(37, 4, 1.5)]

_refs = {}


def _ref(prob):
    if prob.name not in _refs:
        _refs[prob.name] = vcycle.Cycle(prob)
    return _refs[prob.name]


def _close(prob, got, want, bits, cycles):
    off = np.abs(got - want).max() / np.abs(want).max()
    n = max(sum(b.nx for b in prob.blocks), sum(b.ny for b in prob.blocks))
    tol = 1e-3 if prob in CORNER else 8.0 * 2.0 ** -bits * n * cycles
    assert off <= tol, (prob.name, cycles, off, tol)


@pytest.mark.parametrize("prob", EVEN + ODD + LDS + CORNER, ids=lambda p: p.name)
def test_cells_of_fp64_cycles(prob):
    import torch
    import paper_2106_03583_amd as m
    print(f"cells fp64 {prob.name}", flush=True)
    ref = _ref(prob)
    f, start, other = W.rhs(prob, 81), 1e-3 * W.rhs(prob, 82), 1e3 * W.rhs(prob, 86)
    fd, sd, od = (torch.from_numpy(a).cuda() for a in (f, start, other))
    for cycles in (1, 2, 3):
        plan = m.Plan(prob, max_cycles=cycles)
        for flags in (0, m.RETIRE, m.WARM_START):
            p = torch.zeros_like(fd)  # (leaves other values in every buffer of the plan)
            plan.solve(od, p, rtol=1e-15, flags=m.PROJECT_RHS | m.RETIRE, raise_on_error=False)
            p = sd.clone()
            plan.solve(fd, p, rtol=1e-15, flags=m.PROJECT_RHS | flags, raise_on_error=False)
            want = ref.solve(f, cycles, start=start if flags & m.WARM_START else None)
            _close(prob, p.cpu().numpy(), want, 53, cycles)
        plan.close()


@pytest.mark.parametrize("inner", [1, 2, 3])
@pytest.mark.parametrize("prob", EVEN + ODD + LDS + CORNER, ids=lambda p: p.name)
def test_cells_of_mixed_cycles(prob, inner):
    import torch
    import paper_2106_03583_amd as m
    print(f"cells mixed {prob.name} {inner}", flush=True)
    f = W.rhs(prob, 83)
    fd, od = torch.from_numpy(f).cuda(), torch.from_numpy(1e3 * W.rhs(prob, 86)).cuda()
    want = _ref(prob).solve(f, 1, inner)
    plan = m.Plan(prob, precision="mixed", max_cycles=1, inner=inner)
    for flags in (0, m.RETIRE):
        p = torch.zeros_like(fd)
        plan.solve(od, p, rtol=1e-15, flags=m.PROJECT_RHS, raise_on_error=False)
        plan.solve(fd, p, rtol=1e-15, flags=m.PROJECT_RHS | flags, raise_on_error=False)
        _close(prob, p.cpu().numpy(), want, 24, inner)
    plan.close()


@pytest.mark.parametrize("inner", [1, 2, 3])
@pytest.mark.parametrize("name,probs", [("even", EVEN), ("odd", EVEN[:2] + ODD)])
def test_cells_of_grouped_cycles(name, probs, inner):
    import torch
    import paper_2106_03583_amd as m
    print(f"cells grouped {name} {inner}", flush=True)
    f = [W.rhs(pr, 84 + i) for i, pr in enumerate(probs)]
    fd = [torch.from_numpy(a).cuda() for a in f]
    plans = [m.Plan(pr, precision="mixed", max_cycles=1, inner=inner) for pr in probs]
    x = [torch.zeros_like(a) for a in fd]
    m.solve_batch(plans, [1e3 * a.flip(0) for a in fd], x, rtol=1e-15, flags=m.PROJECT_RHS, raise_on_error=False)
    m.solve_batch(plans, fd, x, rtol=1e-15, flags=m.PROJECT_RHS, raise_on_error=False)
    for pr, a, b in zip(probs, f, x):
        _close(pr, b.cpu().numpy(), _ref(pr).solve(a, 1, inner), 24, inner)
    for pl in plans:
        pl.close()
