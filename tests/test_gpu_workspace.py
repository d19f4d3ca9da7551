"""plan_check's workspace covers what the plan allocates, so a server whose budget is sized
with it takes the request: planes around the sizes where the LDS-resident levels' tables
outweigh the buffers they save (few modes, up to 4096 cells in LDS)."""
import pytest

import oracle
import workloads as W
from test_gpu_pair import _box

pytestmark = pytest.mark.gpu

PROBLEMS = [_box(16, 128, "DD", "NN", nz=2), _box(32, 96, "NN", "DD", nz=2), _box(64, 64, "DD", "NN", nz=2),
            _box(48, 64, "DD", "PP", nz=4), _box(128, 96, "DD", "NN", nz=2), W.lshape(32, 2, 1.2)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("prob", PROBLEMS, ids=lambda p: p.name)
def test_a_checked_budget_is_enough(prob, precision):
    import torch
    import paper_2106_03583_amd as m
    inner = 2 if precision == "mixed" else 0  # (the server's default)
    said = m.plan_check(prob, precision=precision, inner=inner)["workspace_bytes"]
    plan = m.Plan(prob, precision=precision, inner=inner)
    assert plan.workspace_bytes <= said
    plan.close()
    f = W.rhs(prob, 11)
    fd = torch.from_numpy(f).cuda()
    p = torch.zeros_like(fd)
    torch.cuda.synchronize()
    srv = m.Server(hbm_budget=said, slots=1, precision=precision)
    status = srv.wait(srv.submit(prob, fd, p, rtol=1e-10, flags=m.PROJECT_RHS))[0]
    srv.close()
    assert status == 0
    assert oracle.rel_error(p.cpu().numpy(), oracle.solve(prob, f)) <= 1e-9
