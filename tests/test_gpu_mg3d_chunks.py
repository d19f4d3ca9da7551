"""The z-marching sweeps of the 3D multigrid where their chunks of planes and
their x-y tiles end unevenly, against the FFT-accelerated path.

A level of 128 tiles is marched over 80 planes in chunks of six with two left
over, over 72 in twelve whole chunks and over 64 in sixteen of four; the
smallest levels have chunks of two planes.  Both solvers stop at a residual of
1e-11 of the right-hand side, above the rounding floor of either, and the bar on
their answers is the solvers' own, 1e-9.
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _cases():
    out = [W.box(512, 256, nz, 8.0, 4.0, nz / 64.0, "DD", "NN", zk, name=f"512x256x{nz}_{zk}")
           for nz, zk in ((64, "PP"), (72, "DD"), (80, "DN"))]
    out.append(W.box(72, 40, 34, 72 / 64, 40 / 64, 34 / 64, "DD", "PP", "NN", name="72x40x34"))
    out.append(W.box(66, 18, 2, 66 / 64, 18 / 64, 2 / 64, "PP", "DD", "PP", name="66x18x2"))
    out.append(W.lshape(72, 36, 1.5, 1.0))
    return out


@pytest.mark.parametrize("prob", _cases(), ids=lambda p: p.name)
def test_mg3d_uneven_chunks(prob):
    import numpy as np
    import torch
    import paper_2106_03583_amd as m
    print(f"mg3d chunks {prob.name}", flush=True)
    f = torch.from_numpy(np.ascontiguousarray(W.rhs(prob, 67))).cuda()
    sols = []
    for plan in (m.Plan3D(prob), m.Plan(prob)):
        p = torch.zeros_like(f)
        info = plan.solve(f, p, rtol=1e-11, flags=m.PROJECT_RHS)
        plan.close()
        assert info.status == 0, info
        sols.append(p)
    a, b = sols
    err = ((a - b).norm() / b.norm()).item()
    print(f"  error {err:.2e}", flush=True)
    assert err <= 1e-9
