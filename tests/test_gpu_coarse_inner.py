"""Mixed problems whose whole hierarchy fits LDS, in a grouped batch: one refinement step
is `inner` FP32 cycles, as when the problem is solved alone, in one launch, whatever the
problems beside it are.

Tolerance as for single cycles: eight roundings a residual times the cells across."""
import numpy as np
import pytest

import vcycle
import workloads as W
from test_gpu_coarse import _ring
from test_gpu_pair import _box

pytestmark = pytest.mark.gpu

PROBLEMS = [_box(64, 64, "DD", "NN"), _box(112, 90, "DD", "NN"), _box(33, 31, "DD", "DN", "ND", fx=1.5), _ring([24, 21, 16], 12),
            _box(40, 36, "NN", "PP", "PP")]


@pytest.mark.parametrize("chosen", [[0], [0, 2, 3, 4], [0, 1, 2, 3, 4]], ids=str)
@pytest.mark.parametrize("inner", [1, 2, 4])
def test_inner_cycles_in_lds(inner, chosen):
    import torch
    import paper_2106_03583_amd as m
    probs = [PROBLEMS[i] for i in chosen]
    f = [W.rhs(p, 91 + i) for i, p in enumerate(probs)]
    fd = [torch.from_numpy(a).cuda() for a in f]
    for cycles in (1, 2):
        plans = [m.Plan(p, precision="mixed", max_cycles=cycles, inner=inner) for p in probs]
        x = [torch.zeros_like(a) for a in fd]
        m.solve_batch(plans, fd, x, rtol=1e-15, flags=m.PROJECT_RHS, raise_on_error=False)
        for p, a, b, pl, r in zip(probs, f, x, plans, fd):
            want = vcycle.Cycle(p).solve(a, cycles, inner)
            alone = torch.zeros_like(b)
            pl.solve(r, alone, rtol=1e-15, flags=m.PROJECT_RHS | m.RETIRE, raise_on_error=False)
            n = max(sum(k.nx for k in p.blocks), sum(k.ny for k in p.blocks))
            for got in (b, alone):
                off = np.abs(got.cpu().numpy() - want).max() / np.abs(want).max()
                assert off <= 8.0 * 2.0 ** -24 * n * inner * cycles, (p.name, cycles, off)
        for pl in plans:
            pl.close()
