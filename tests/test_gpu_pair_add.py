"""Mixed solves whose last FP32 sweep adds straight to the FP64 iterate, with one,
two and three inner cycles (from a zero correction and from a stored one, in
either buffer), in the retiring, lockstep, warm-started and batched forms; the batch
holds a plane that the march does not take and adds in a pass of its own.

Tolerances as for the march itself: rtol 1e-10 bounds the 3D residual, 10 rtol the
relative error."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_pair import PROBLEMS, _box

pytestmark = pytest.mark.gpu
CASES = [PROBLEMS[2], PROBLEMS[7], PROBLEMS[13], PROBLEMS[16]]


def _check(prob, ref, fproj, p):
    got = p.cpu().numpy()
    assert oracle.rel_residual(prob, got, fproj) <= 1e-10
    assert oracle.rel_error(got, ref) <= 1e-9


@pytest.mark.parametrize("inner", [1, 2, 3])
def test_pair_add(inner):
    import torch
    import paper_2106_03583_amd as m
    probs = CASES + [_box(113, 92, "DD", "NN")]
    f = [W.rhs(pr, 42) for pr in probs]
    ref = [oracle.solve(pr, x) for pr, x in zip(probs, f)]
    fp = [oracle.project_compatible(pr, x) if oracle.is_singular(pr) else x for pr, x in zip(probs, f)]
    plans = [m.Plan(pr, precision="mixed", inner=inner) for pr in probs]
    fd = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in f]
    for i, pr in enumerate(probs):
        print(f"pair add {pr.name} inner={inner}", flush=True)
        for flags in (0, m.RETIRE, m.RETIRE | m.WARM_START):
            p = torch.from_numpy(0.5 * ref[i]).cuda() if flags & m.WARM_START else torch.zeros_like(fd[i])
            plans[i].solve(fd[i], p, rtol=1e-10, flags=m.PROJECT_RHS | flags)
            _check(pr, ref[i], fp[i], p)
    for chosen in (range(len(CASES)), range(len(probs))):  # without and with the other plane
        ps = [torch.zeros_like(fd[i]) for i in chosen]
        m.solve_batch([plans[i] for i in chosen], [fd[i] for i in chosen], ps, rtol=1e-10, flags=m.PROJECT_RHS)
        for i, p in zip(chosen, ps):
            _check(probs[i], ref[i], fp[i], p)
    for pl in plans:
        pl.close()
