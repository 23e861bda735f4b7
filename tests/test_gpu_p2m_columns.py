"""P2M of lattice sources and its transpose on meshes of few octets with many
models, whose blocks of 16 columns hold several models: octets in and out of
the M2L's reach, leaves at level 2 and below, one and two parts of the rows.

Bars: a batch against its models one by one, which differ in the order of the
M2L's sums alone: 1e-12 FP64, FP32 M2L 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


@pytest.mark.parametrize("prec, bar", [(G.GRAV_FP64, 1e-12), (G.GRAV_MIXED, 1e-5)], ids=["fp64", "mixed"])
@pytest.mark.parametrize("p", [5, 10, 14])
@pytest.mark.parametrize("n, batch", [((16, 4, 4), 37), ((13, 9, 30), 7), ((4, 4, 70), 5), ((1, 1, 1), 50), ((24, 24, 24), 2)])
def test_p2m_columns(n, batch, p, prec, bar):
    pts = np.random.default_rng(p).uniform(0.0, 1.0, size=(20, 3)) * np.array([5.0, 4.0, 1.0]) + [0.0, 0.0, n[2] + 8.0]

    def plan(b):
        return G.Plan(G.PlanSpec(n=n, h=1.0, voxel_centres=False, components=3, p=p, leaf_size=64, points=pts,
                                 precision=prec, batch=b))

    one, many = plan(1), plan(batch)
    assert many.levels >= 2 and many.check() == "ok"
    gen = torch.Generator(device="cuda").manual_seed(p)
    rho = torch.rand(many.rho_shape, dtype=torch.float64, device="cuda", generator=gen) + 0.1
    g = many.eval(rho)
    ref = torch.stack([one.eval(rho[b].contiguous()) for b in range(batch)])
    assert float((g - ref).norm() / ref.norm()) <= bar
    r = torch.randn(many.out_shape, dtype=torch.float64, device="cuda", generator=gen)
    d = many.adjoint(r)
    ref = torch.stack([one.adjoint(r[b].contiguous()) for b in range(batch)])
    assert float((d - ref).norm() / ref.norm()) <= bar
