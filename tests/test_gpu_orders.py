"""Truncation error of every expansion order, which a wrong coefficient of any
degree would change: leaves of one and of 4^3 cells with cell centres and points,
and scattered sources with points.

Bars: the errors (phi, g; relative L2 against the direct sum) were measured with
kernels that sum over the offsets of single boxes, and hold to 1e-3 of each: the
truncated sums are the same, only rounding differs.  Mixed plans differ from
FP64 ones by FP32 rounding, 1e-5."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")

ERRORS = {
    "cells of 1": [4.7825e-01, 1.0212e-01, 2.5707e-02, 7.8939e-03, 2.5574e-03, 8.2869e-04, 3.1517e-04, 1.1861e-04,
                   4.5793e-05, 1.9116e-05, 7.9828e-06, 3.3891e-06, 1.3825e-06, 7.0794e-07, 2.6999e-07, 1.4279e-07],
    "cells of 64": [2.2599e-01, 6.9061e-02, 2.3137e-02, 7.9622e-03, 2.6785e-03, 1.0602e-03, 4.1112e-04, 1.6503e-04,
                    6.8114e-05, 2.9062e-05, 1.1878e-05, 4.9355e-06, 2.3310e-06, 1.1301e-06, 5.5032e-07, 2.7006e-07],
    "scattered": [7.0136e-02, 1.4086e-02, 5.3662e-03, 1.8111e-03, 7.1348e-04, 2.8612e-04, 1.2519e-04, 5.7974e-05,
                  2.6853e-05, 1.1155e-05, 6.5313e-06, 1.6876e-06, 1.0038e-06, 5.4923e-07, 4.3768e-07, 1.0803e-07],
}


@pytest.mark.parametrize("p", range(1, 17))
@pytest.mark.parametrize("kind", list(ERRORS))
def test_truncation_error(kind, p):
    rng = np.random.default_rng(3)
    if kind == "cells of 1":
        spec = dict(n=(19, 16, 13), leaf_size=1, voxel_centres=True, points=rng.uniform(-0.3, 1.4, size=(60, 3)))
    elif kind == "cells of 64":
        spec = dict(n=(37, 30, 26), leaf_size=64, voxel_centres=True, points=rng.uniform(-0.3, 2.4, size=(60, 3)))
    else:
        spec = dict(n=(24, 24, 24), leaf_size=64, voxel_centres=False, points=rng.uniform(0.0, 1.5, size=(900, 3)),
                    sources=rng.uniform(0.0, 1.5, size=(4000, 3)))
    f64, mixed = (G.Plan(G.PlanSpec(h=1 / 16, components=4, p=p, precision=prec, **spec))
                  for prec in (G.GRAV_FP64, G.GRAV_MIXED))
    rho = torch.as_tensor(np.random.default_rng(p).normal(size=f64.rho_shape), device="cuda")
    if kind == "scattered":
        exact = torch.as_tensor(oracle.points(spec["sources"], rho.cpu().numpy(), spec["points"]), device="cuda")
    else:
        exact = f64.direct(rho)
    out = f64.eval(rho)
    exact = exact.reshape(out.shape)
    e, bar = float((out - exact).norm() / exact.norm()), ERRORS[kind][p - 1]
    assert abs(e - bar) <= 1e-3 * bar
    assert float((mixed.eval(rho) - out).norm() / out.norm()) <= 1e-5
