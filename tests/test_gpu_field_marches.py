"""The z-marching kernels on the packed fields (operator, residual check, velocity
correction) where tiles of 64 x 16 and chunks of planes end unevenly, against the
oracle.

One cell wider and narrower than a tile, rows that leave a partial row group,
blocks joined across ragged edges, and a plane of 128 tiles whose 70 planes are
marched in chunks of six with four left over.  Each result is a sum of at most
ten products no larger than a few times the largest result, so 1e-12 of that is
some thousand roundings.
"""
import numpy as np
import pytest

import oracle
import oracle.projection as PJ
import workloads as W

pytestmark = pytest.mark.gpu


def _cases():
    out = [W.box(nx, ny, nz, nx / 64, ny / 64, nz / 64, xp, yp, zp, xfactor=1.1, name=f"{nx}x{ny}x{nz}_{xp}{yp}{zp}")
           for nx, ny, nz, xp, yp, zp in ((63, 15, 4, "DN", "PP", "PP"), (64, 16, 6, "PP", "ND", "DD"),
                                          (65, 17, 10, "NN", "DD", "ND"), (130, 35, 2, "DD", "NN", "DN"),
                                          (512, 256, 70, "DN", "NN", "NN"))]
    return out + [W.lshape(36, 8, 1.5, 1.0), W.random_layout(11), W.random_layout(100)]


@pytest.mark.parametrize("prob", _cases(), ids=lambda p: p.name)
def test_field_marches(prob):
    import torch
    import paper_2106_03583_amd as m
    print(f"marches {prob.name}", flush=True)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    rng = np.random.default_rng(5)
    plan = m.Plan(prob, helmholtz=0.5)
    p, f = rng.standard_normal(plan.ncells), rng.standard_normal(plan.ncells)
    ref = oracle.apply_3d(oracle.Geometry(prob), p, 0.5)
    out = torch.full((plan.ncells,), float("nan"), dtype=torch.float64, device="cuda")
    plan.apply(dev(p), out)
    assert np.abs(out.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
    norms = plan.residual_norm(dev(f), dev(p), 0.25).cpu().numpy()
    expect = [np.linalg.norm(f - 0.25 - ref), np.linalg.norm(f - 0.25)]
    assert np.allclose(norms, expect, rtol=1e-12, atol=0)
    plan.close()

    plan = m.Plan(prob)
    uvw = PJ.make_consistent(prob, *(rng.standard_normal(n) for n in PJ.face_sizes(prob)))
    new = [dev(a) for a in uvw]
    phi = torch.zeros(plan.ncells, dtype=torch.float64, device="cuda")
    # the correction alone is compared, so how far the solve gets does not matter
    plan.project(*new, 0.05, phi, torch.empty_like(phi), rtol=1e-3, flags=m.PROJECT_RHS)
    for a, g, b in zip(uvw, PJ.gradient(prob, phi.cpu().numpy()), new):
        exp = a - 0.05 * g
        assert np.abs(b.cpu().numpy() - exp).max() <= 1e-12 * max(np.abs(exp).max(), 0.05 * np.abs(g).max())
    plan.close()
