"""The plan tuner times candidates only where they differ: on the strip kernels' levels.  A
plan whose levels run the pair march or in LDS has one schedule, timed once."""
import pytest

import workloads as W
from test_gpu_strips import MARCHED, STRIPS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("prob,strips", [(STRIPS[0], True), (MARCHED[0], False), (MARCHED[1], False)],
                         ids=lambda v: getattr(v, "name", ""))
def test_tuner_times_what_differs(prob, strips, precision):
    import torch
    import paper_2106_03583_amd as m
    fd = torch.from_numpy(W.rhs(prob, 24)).cuda()
    plan = m.Plan(prob, precision=precision, inner=1)
    plan.profile(True)
    t = plan.autotune(fd)
    sweeps = max(plan.profile_read()["launches"])
    plan.profile(False)
    assert 0.0 < t["ms_tuned"] <= t["ms_default"]
    if strips:
        assert sweeps > 4
    else:  # one schedule: one warm-up and three timed cycles
        assert sweeps == 4 and t["ms_tuned"] == t["ms_default"]
        assert t["wg_target"] == 768 and not any(t["form"])
    p = torch.zeros_like(fd)
    assert plan.solve(fd, p, rtol=1e-10, flags=m.PROJECT_RHS | m.RETIRE).status == 0
    plan.close()
