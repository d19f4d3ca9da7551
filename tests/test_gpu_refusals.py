"""A refused right-hand side costs no cycle: nothing that is queued behind the checks finds
an active mode, whatever the form of the solve, and the report says so."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_pair import _box

pytestmark = pytest.mark.gpu

# marched, whole hierarchy in LDS, in LDS with a step that halves x alone
PROBLEMS = [_box(96, 80, "NN", "NN", "NN"), _box(40, 36, "NN", "PP", "PP"),
            W.box(48, 20, 6, 0.25, 0.5, 0.1, "NN", "NN", "NN", name="48x20_flat")]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("prob", PROBLEMS, ids=lambda p: p.name)
def test_refused_solves_run_no_cycle(prob, precision):
    import torch
    import paper_2106_03583_amd as m
    good = oracle.project_compatible(prob, W.rhs(prob, 37))
    nan = good.copy()
    nan[len(nan) // 2] = np.nan
    plan = m.Plan(prob, precision=precision)
    p = torch.zeros(prob.ncells, dtype=torch.float64, device="cuda")
    for flags in (0, m.RETIRE, m.RETIRE | m.WARM_START):
        for f, extra, want in ((nan, 0, m.ERR_NONFINITE), (nan, m.PROJECT_RHS, m.ERR_NONFINITE),
                               (good + 1.0, 0, m.ERR_INCOMPATIBLE)):
            p.fill_(3.0)
            info = plan.solve(torch.from_numpy(f).cuda(), p, flags=flags | extra, raise_on_error=False)
            assert info.status == want
            assert info.cycles == 0 and not info.cycles_per_mode.any()
            assert float((p - 3.0).abs().max()) == 0.0
        p.zero_()
        info = plan.solve(torch.from_numpy(good).cuda(), p, rtol=1e-10, flags=flags)
        assert info.status == 0 and info.cycles > 0
        assert oracle.rel_error(p.cpu().numpy(), oracle.solve(prob, good)) <= 1e-9
    plan.close()
