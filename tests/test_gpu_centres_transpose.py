"""Transposed far-field evaluation at the centres of 4^3-cell leaves: every
number of class row blocks and components, ragged blocks of leaves, leaves that
hold user points too, several models.

Bar: the transpose identity to FP64 rounding, 1e-12."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


@pytest.mark.parametrize("p", [1, 4, 9, 11, 16])
@pytest.mark.parametrize("comps", [1, 3, 4])
def test_centres_transpose(p, comps):
    pts = np.random.default_rng(p).uniform(0.0, 1.0, size=(30, 3)) * np.array([37.0, 22.0, 18.0])
    plan = G.Plan(G.PlanSpec(n=(37, 22, 18), h=1.0, voxel_centres=True, components=comps, p=p, leaf_size=64, points=pts,
                             precision=G.GRAV_FP64, batch=2))
    gen = torch.Generator(device="cuda").manual_seed(p)
    rho = torch.randn(plan.rho_shape, dtype=torch.float64, device="cuda", generator=gen)
    r = torch.randn(plan.out_shape, dtype=torch.float64, device="cuda", generator=gen)
    g, d = plan.eval(rho), plan.adjoint(r)
    gap = abs(float((g * r).sum()) - float((rho * d).sum())) / (float(g.norm()) * float(r.norm()))
    assert gap <= 1e-12
