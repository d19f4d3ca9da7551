"""Checks of the rhs, whose values reach the host through memory that kernels write: plans
and server slots pass from good to refused right-hand sides and back, many times over, and
every solve gets the status of its own rhs, never of the one before."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_pair import _box

pytestmark = pytest.mark.gpu

SINGULAR = [_box(96, 80, "NN", "NN", "NN"), _box(40, 36, "NN", "PP", "PP")]  # marched; whole hierarchy in LDS


def _inputs(m, prob):
    good = oracle.project_compatible(prob, W.rhs(prob, 31))
    nan, inc = good.copy(), good + 1.0
    nan[-1] = np.inf
    return [(good, 0), (nan, m.ERR_NONFINITE), (good, 0), (inc, m.ERR_INCOMPATIBLE), (nan, m.ERR_NONFINITE),
            (inc, m.ERR_INCOMPATIBLE)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("prob", SINGULAR, ids=lambda p: p.name)
def test_status_of_its_own_rhs(prob, precision):
    import torch
    import paper_2106_03583_amd as m
    print(f"checks {prob.name} {precision}", flush=True)
    plan = m.Plan(prob, precision=precision)
    cases = [(torch.from_numpy(f).cuda(), st) for f, st in _inputs(m, prob)]
    p = torch.zeros_like(cases[0][0])
    for n in range(30):
        for f, want in cases:
            p.fill_(3.0)
            info = plan.solve(f, p, rtol=1e-8, flags=m.RETIRE if n & 1 else 0, raise_on_error=False)
            assert info.status == want
            assert (float((p - 3.0).abs().max()) == 0.0) == (want != 0)
    plan.close()


def test_status_of_its_own_request():
    import torch
    import paper_2106_03583_amd as m
    srv = m.Server(hbm_budget=1 << 30, slots=2, precision="mixed")
    cases = [(pr, torch.from_numpy(f).cuda(), st) for pr in SINGULAR for f, st in _inputs(m, pr)]
    outs = [torch.zeros_like(f) for _, f, _ in cases]
    torch.cuda.synchronize()
    for _ in range(10):
        tickets = [srv.submit(pr, f, o, rtol=1e-8) for (pr, f, _), o in zip(cases, outs)]
        assert [srv.wait(t)[0] for t in tickets] == [st for _, _, st in cases]
    srv.close()
