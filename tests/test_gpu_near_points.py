"""Near field of user points: cells of the 27 leaves in one and several chunks,
1- and 2-point rules, scattered sources (with empty leaves) at leaves of up to
16 points, in and out of whole groups of four, and of more, several models.

Bar: a leaf edge that leaves no far field (one leaf, or levels 0 and 1) makes
the FMM the direct sum: 1e-12 FP64, FP32 pairs 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


@pytest.mark.parametrize("prec", [G.GRAV_FP64, G.GRAV_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("npts", [1, 6, 16, 17, 300])
@pytest.mark.parametrize("kind", ["cells", "cells2", "sources"])
def test_near_points(kind, npts, prec):
    rng = np.random.default_rng(npts)
    n = (16, 9, 13)
    pts = np.concatenate([rng.uniform(0.0, 7.9, size=(npts, 3)), [[15.5, 8.5, 12.5]], [[8.0, 4.0, 6.5]]])
    src = dict(sources=rng.uniform(0.0, 1.0, size=(700, 3)) * np.array([16.0, 9.0, 4.0])) if kind == "sources" else {}
    plan = G.Plan(G.PlanSpec(n=n, h=1.0, voxel_centres=False, components=4, p=4, leaf_size=512 * (8 if kind == "cells2" else 1),
                             quad_order=2 if kind == "cells2" else 1, points=pts, precision=prec, batch=2, **src))
    assert plan.levels < 2
    gen = torch.Generator(device="cuda").manual_seed(npts)
    rho = torch.randn(plan.rho_shape, dtype=torch.float64, device="cuda", generator=gen)
    g = plan.eval(rho)
    if kind == "sources":  # (phi, g) = sum of m (1 / r, (t - x) / r^3)
        d = torch.tensor(pts[:, None] - src["sources"][None], device="cuda")
        ri = d.norm(dim=2).reciprocal()
        k = torch.cat([ri[..., None], d * ri[..., None] ** 3], 2)
        ref = (rho.reshape(2, 1, -1, 1) * k[None]).sum(2)
    else:
        ref = plan.direct(rho)
    assert float((g - ref).norm() / ref.norm()) <= (1e-12 if prec == G.GRAV_FP64 else 1e-5)
