"""The two forms of a batched solve and sets that need both: FP64 problems alone, FP64
beside mixed ones, mixed problems off the group (an odd ring on a global level, another
inner cycle count, two sweeps), one problem alone, problems that end at once or are
refused, and whole hierarchies in LDS; with and without tuning, again on the same plans,
and from a warm start.  Bounds: rtol on the residual, 10 rtol on the error, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_pair import C, D, N, _box, _grid

pytestmark = pytest.mark.gpu

ODD = W.box(302, 256, 4, 302 / 128, 2.0, 4 / 128, "PP", "NN", "DD", name="odd302")
BIG = [_box(112, 90, "DD", "NN"), _box(203, 157, "ND", "DD", "NN"), _grid([56, 60], [40, 64], [(1, 1)], [N, D]),
       _box(96, 160, "NN", "PP", "DD"), _box(130, 66, "NN", "NN", "DN")]
LDS = [_box(64, 64, "NN", "PP", "DN"), _box(48, 32, "ND", "DN")]

SETS = {
    "fp64": [(p, "fp64", {}) for p in BIG + LDS],
    "fp64_one": [(BIG[1], "fp64", {})],
    "both": [(BIG[0], "fp64", {}), (BIG[1], "mixed", {}), (LDS[0], "fp64", {}), (BIG[2], "mixed", {}), (BIG[3], "fp64", {}),
             (LDS[1], "mixed", {})],
    "off_group": [(BIG[0], "mixed", {}), (ODD, "mixed", {}), (BIG[1], "mixed", {"inner": 2}),
                  (BIG[3], "mixed", {"nu1": 2, "nu2": 2}), (BIG[2], "mixed", {})],
    "lds_only": [(p, "fp64", {}) for p in LDS],
    "grouped": [(p, "mixed", {}) for p in BIG + LDS],
}


@pytest.mark.parametrize("name", list(SETS))
def test_batch_forms(name):
    import torch
    import paper_2106_03583_amd as m
    print(f"batch forms {name}", flush=True)
    probs = [p for p, _, _ in SETS[name]]
    plans = [m.Plan(p, precision=prec, **kw) for p, prec, kw in SETS[name]]
    for n, flags in enumerate((0, m.AUTOTUNE, 0, m.WARM_START)):
        f = [W.rhs(p, 70 + 10 * n + i) for i, p in enumerate(probs)]
        fd = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in f]
        if flags & m.WARM_START:
            x = [torch.from_numpy(0.5 * oracle.solve(p, a)).cuda() for p, a in zip(probs, f)]
        else:
            x = [torch.full_like(a, float("nan")) for a in fd]
        infos = m.solve_batch(plans, fd, x, rtol=1e-10, flags=m.PROJECT_RHS | flags)
        for p, a, b, info in zip(probs, f, x, infos):
            assert info.status == 0 and info.cycles == max(info.cycles_per_mode)
            fp = oracle.project_compatible(p, a) if oracle.is_singular(p) else a
            assert oracle.rel_residual(p, b.cpu().numpy(), fp) <= 1e-10
            assert oracle.rel_error(b.cpu().numpy(), oracle.solve(p, a)) <= 1e-9
    if name != "lds_only":  # streams: 0 where every problem was grouped
        assert (m.batch_schedule(plans)[0] == 0) == (name == "grouped")
    for pl in plans:
        pl.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch_ends_and_refusals(precision):
    """A zero rhs (no cycle), a NaN, an incompatible one and a cycle limit, beside a good one."""
    import torch
    import paper_2106_03583_amd as m
    probs = [BIG[0], BIG[0], BIG[0], _box(90, 70, "NN", "NN", "NN"), BIG[1]]
    plans = [m.Plan(p, precision=precision, max_cycles=2 if i == 4 else 100) for i, p in enumerate(probs)]
    f = [W.rhs(p, 90 + i) for i, p in enumerate(probs)]
    f[1] = np.zeros_like(f[1])
    f[2][5] = np.nan
    f[3] = f[3] + 1.0
    fd = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in f]
    for _ in range(2):
        x = [torch.full_like(a, 7.0) for a in fd]
        infos = m.solve_batch(plans, fd, x, rtol=1e-10, flags=0, raise_on_error=False)
        assert [i.status for i in infos] == [0, 0, m.ERR_NONFINITE, m.ERR_INCOMPATIBLE, m.ERR_NOT_CONVERGED]
        assert [i.cycles for i in infos[1:]] == [0, 0, 0, 2]
        assert oracle.rel_error(x[0].cpu().numpy(), oracle.solve(probs[0], f[0])) <= 1e-9
        assert float(x[1].abs().max()) == 0.0
        assert float((x[2] - 7.0).abs().max()) == 0.0 and float((x[3] - 7.0).abs().max()) == 0.0
    for pl in plans:
        pl.close()
