"""z transforms over the lengths where the wide kernel's plan changes, against the
oracle's dense basis.

Between them the half lengths use every stage radix (2 to 10, 12, 15, 16) with one
to several stages, are odd and even, give tiles of 64, 32, 16 and 8 columns with
threads left over, and leave the last pass of rows, the last tile of a block and
the last tile of a workgroup's loop incomplete; 34 and 1122 (primes above 7) and
2048 with the cosine kinds (no room for the tables) stay with the per-tile kernel.
The bound is that of the other transform tests: 1e-12 sqrt(n) of the largest value.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_parity import two_block

pytestmark = pytest.mark.gpu

LENGTHS = [2, 4, 6, 14, 18, 30, 34, 54, 90, 98, 144, 150, 250, 270, 300, 360, 384, 486, 490, 640, 686, 720, 1000, 1050, 1122,
           1152, 1296, 2048]


def _check(torch, m, prob, kind, nz):
    plan = m.Plan(prob)
    g, T = oracle.Geometry(prob), oracle.basis(kind, nz)
    x = np.random.default_rng(nz).standard_normal(plan.ncells)
    out = torch.full((plan.ncells,), float("nan"), dtype=torch.float64, device="cuda")
    tol = 1e-12 * np.sqrt(nz)
    plan.forward(torch.from_numpy(x).cuda(), out)
    ref = np.concatenate([T.T @ b.reshape(nz, -1) for b in g.split3(x)], axis=1)
    assert np.abs(out.cpu().numpy().reshape(nz, -1) - ref).max() <= tol * np.abs(ref).max()
    out.fill_(float("nan"))
    plan.inverse(torch.from_numpy(x).cuda(), out)
    xm = x.reshape(nz, -1)
    ref = np.concatenate([(T @ xm[:, g.off2[i]:g.off2[i + 1]]).ravel() for i in range(g.nb)])
    assert np.abs(out.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
    plan.close()


@pytest.mark.parametrize("kind", ["PP", "NN", "DD", "ND", "DN"])
@pytest.mark.parametrize("nz", LENGTHS)
def test_transform_lengths(kind, nz):
    import torch
    import paper_2106_03583_amd as m
    print(f"transform {kind} nz={nz}", flush=True)
    _check(torch, m, two_block(nz, kind, 16, 6, 9), kind, nz)
    if nz in (90, 270, 300):  # several tiles a workgroup, the last incomplete
        _check(torch, m, two_block(nz, kind, 161, 63, 67), kind, nz)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("kind,nz", [("PP", 512), ("NN", 90), ("DN", 270)])
def test_not_finite_is_seen(kind, nz, bad):
    import torch
    import paper_2106_03583_amd as m
    prob = two_block(nz, kind, 16, 6, 9)
    plan = m.Plan(prob)
    f = torch.from_numpy(W.rhs(prob, 3)).cuda()
    f[-1] = bad
    info = plan.solve(f, torch.zeros_like(f), rtol=1e-8, raise_on_error=False)
    plan.close()
    assert info.status == m.ERR_NONFINITE
