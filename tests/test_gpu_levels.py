"""Translations between levels over sibling octets: the kernels of wide levels
(a dozen models on a ragged mesh: 9072 columns on the leaf level, no multiple
of the column blocks of the level above) against those of narrow ones (the
same models one by one), both directions.

Bars: the two differ in the order of sums alone, so rounding (1e-12 FP64; FP32
M2L and near field 1e-5)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


def _plan(p, prec, batch, centres):
    return G.Plan(G.PlanSpec(n=(46, 34, 27), h=1 / 16, voxel_centres=centres, components=3, p=p, leaf_size=2,
                             points=np.random.default_rng(3).uniform(0.0, 2.0, size=(60, 3)), precision=prec,
                             batch=batch))


@pytest.mark.parametrize("centres", [True, False], ids=["volume", "stations"])
@pytest.mark.parametrize("p, prec", [(5, G.GRAV_FP64), (10, G.GRAV_FP64), (16, G.GRAV_FP64), (10, G.GRAV_MIXED)])
def test_wide_levels(p, prec, centres):
    bar = 1e-12 if prec == G.GRAV_FP64 else 1e-5
    one, many = _plan(p, prec, 1, centres), _plan(p, prec, 12, centres)
    assert many.check() == "ok"
    gen = torch.Generator(device="cuda").manual_seed(p)
    rho = torch.randn(many.rho_shape, dtype=torch.float64, device="cuda", generator=gen)
    g = many.eval(rho)
    ref = torch.stack([one.eval(rho[b].contiguous()) for b in range(12)])
    assert float((g - ref).norm() / ref.norm()) <= bar
    r = torch.randn(many.out_shape, dtype=torch.float64, device="cuda", generator=gen)
    d = many.adjoint(r)
    ref = torch.stack([one.adjoint(r[b].contiguous()) for b in range(12)])
    assert float((d - ref).norm() / ref.norm()) <= bar
