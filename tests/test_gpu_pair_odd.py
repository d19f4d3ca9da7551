"""The pair march on planes with odd counts (a last coarse cell of three children),
in x, in y and in both: single strips and several, the lone column in a strip of its
own pair and in a halo, strips of rows that end on the odd row, both places of the
middle child against its coarse cell (stretching either way), walls of both
kinds, joined blocks whose odd side ends at a wall, and odd sides at a joined face
or a ring, which the march leaves to the strip kernels.

Tolerances as for the even planes: rtol 1e-10 bounds the 3D residual, 10 rtol the
relative error."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_pair import D, N, _box, _grid

pytestmark = pytest.mark.gpu

PROBLEMS = [
    _box(113, 96, "DD", "NN"), _box(112, 91, "ND", "DD"), _box(111, 97, "NN", "DN", "NN"),
    _box(119, 129, "DN", "ND", fx=1.2), _box(121, 65, "ND", "DD", "DN", fx=-1.2, fy=1.5),
    _box(225, 49, "DD", "NN", "DD", fy=-1.5), _box(241, 131, "NN", "DD", fx=0.7), _box(75, 81, "DD", "PP"),
    _box(9, 1101, "DD", "NN"), _box(1101, 9, "NN", "ND"), _box(67, 259, "DD", "NN", "PP", fx=1.8, fy=1.8),
    _grid([56, 61], [40, 65], [(1, 1)], [N, D]), _grid([60, 8, 57], [36, 49], [], [D, N, N]),
    _grid([57, 60], [40, 64], [], [D, N]), _box(75, 82, "PP", "DD"),
]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("prob", PROBLEMS, ids=lambda p: p.name)
def test_pair_odd(prob, precision):
    import torch
    import paper_2106_03583_amd as m
    print(f"pair odd {prob.name} {precision}", flush=True)
    f = W.rhs(prob, 43)
    ref = oracle.solve(prob, f)
    fproj = oracle.project_compatible(prob, f) if oracle.is_singular(prob) else f
    plan = m.Plan(prob, precision=precision)
    fd = torch.from_numpy(np.ascontiguousarray(f)).cuda()
    for flags in (0, m.RETIRE, m.RETIRE | m.WARM_START):
        p = torch.from_numpy(0.5 * ref).cuda() if flags & m.WARM_START else torch.zeros_like(fd)
        plan.solve(fd, p, rtol=1e-10, flags=m.PROJECT_RHS | flags)
        got = p.cpu().numpy()
        assert oracle.rel_residual(prob, got, fproj) <= 1e-10
        assert oracle.rel_error(got, ref) <= 1e-9
    plan.close()


@pytest.mark.parametrize("inner", [1, 4])
def test_pair_odd_batch(inner):
    """Odd and even planes in one launch."""
    import torch
    import paper_2106_03583_amd as m
    probs = [PROBLEMS[2], _box(114, 92, "NN", "DD", "DD"), PROBLEMS[11], PROBLEMS[14], PROBLEMS[10]]
    plans = [m.Plan(p, precision="mixed", inner=inner) for p in probs]
    f = [torch.from_numpy(np.ascontiguousarray(W.rhs(p, 44))).cuda() for p in probs]
    x = [torch.zeros_like(a) for a in f]
    m.solve_batch(plans, f, x, rtol=1e-10, flags=m.PROJECT_RHS)
    for pr, a, b in zip(probs, f, x):
        fh = a.cpu().numpy()
        fp = oracle.project_compatible(pr, fh) if oracle.is_singular(pr) else fh
        assert oracle.rel_residual(pr, b.cpu().numpy(), fp) <= 1e-10
        assert oracle.rel_error(b.cpu().numpy(), oracle.solve(pr, fh)) <= 1e-9
