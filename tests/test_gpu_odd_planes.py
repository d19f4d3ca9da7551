"""FP64 solves on planes with an odd number of cells, stopped after one, two or three
V-cycles: the modes' iterates then lie in either buffer of the march, and every cell of
the field, the last of each plane included, must be the iterate of that very cycle.  The
plan has solved another problem before, so a cell nobody wrote shows.

Tolerance: rounding, amplified by the square of the cells across (vcycle.tolerance)."""
import numpy as np
import pytest

import vcycle
import workloads as W
from test_gpu_pair import D, N, _box, _grid

pytestmark = pytest.mark.gpu

PROBLEMS = [_box(111, 97, "NN", "DN", "NN"), _box(203, 157, "ND", "DD", "NN"), _box(75, 81, "DD", "ND", "DD", fx=1.1),
            _grid([60, 57], [64, 41], [], [D, N])]


@pytest.mark.parametrize("prob", PROBLEMS, ids=lambda p: p.name)
def test_every_cell_is_the_last_iterate(prob):
    import torch
    import paper_2106_03583_amd as m
    print(f"odd plane {prob.name}", flush=True)
    f, g = W.rhs(prob, 51), 1e3 * W.rhs(prob, 52)
    ref = vcycle.Cycle(prob)
    fd, gd = torch.from_numpy(f).cuda(), torch.from_numpy(g).cuda()
    for cycles in (1, 2, 3):
        want = ref.solve(f, cycles)
        plan = m.Plan(prob, max_cycles=cycles)
        for flags in (0, m.RETIRE):
            p = torch.zeros_like(fd)
            plan.solve(gd, p, rtol=1e-15, flags=m.PROJECT_RHS | flags, raise_on_error=False)
            p.fill_(float("nan"))
            info = plan.solve(fd, p, rtol=1e-15, flags=m.PROJECT_RHS | flags, raise_on_error=False)
            assert info.cycles == cycles
            assert set(info.cycles_per_mode) == {cycles}
            off = np.abs(p.cpu().numpy() - want).max() / np.abs(want).max()
            assert off <= vcycle.tolerance(prob, 53, cycles), (cycles, flags, off)
        plan.close()


def test_one_cycle_meets_a_loose_tolerance():
    """Modes that pass after one V-cycle, retired beside others that need more."""
    import torch
    import paper_2106_03583_amd as m
    prob = _box(111, 97, "DD", "DN", "NN", nz=8)
    f, g = W.rhs(prob, 53), 1e3 * W.rhs(prob, 54)
    plan = m.Plan(prob, helmholtz=2e4, etol=-1.0)
    ref = vcycle.Cycle(prob, alpha=2e4)
    fd, gd = torch.from_numpy(f).cuda(), torch.from_numpy(g).cuda()
    p = torch.zeros_like(fd)
    for rtol in (0.3, 0.05, 0.01, 1e-3, 1e-5):
        plan.solve(gd, p, rtol=1e-8, flags=m.RETIRE)
        info = plan.solve(fd, p, rtol=rtol, flags=m.RETIRE)
        cyc = np.asarray(info.cycles_per_mode)
        want = np.zeros_like(f)
        for c in set(cyc):  # each mode as it was when it retired
            x = ref.modes(ref.solve(f, int(c)))
            x[cyc != c] = 0.0
            want += ref.field(x)
        off = np.abs(p.cpu().numpy() - want).max() / np.abs(want).max()
        print(f"  rtol {rtol}: cycles {sorted(set(cyc))}, off {off:.2e}", flush=True)
        assert off <= vcycle.tolerance(prob, 53, int(cyc.max()))
    plan.close()
