"""M2L over sibling octets: every expansion order (chunks of 1, 3, 4, 5 and 7
k steps, full and short last row blocks, one and two row parts), single and
several column blocks per wave, both precisions and both directions, on a
ragged mesh whose edge octets lack children and sources.

Bars: the FMM against the direct sum within 2 x 0.55^p (one-box separation
converges like 0.4 .. 0.5 per order); the same plan alone and in a batch (other
unit widths and sums) and the transpose to rounding (1e-12 FP64; FP32 M2L and
near field 1e-5)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


def _plan(p, prec, batch):
    return G.Plan(G.PlanSpec(n=(19, 16, 13), h=1 / 16, voxel_centres=True, components=3, p=p, leaf_size=1,
                             points=np.random.default_rng(3).uniform(-0.3, 1.4, size=(60, 3)), precision=prec,
                             batch=batch))


@pytest.mark.parametrize("prec", [G.GRAV_FP64, G.GRAV_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("p", range(1, 17))
def test_octet_m2l(p, prec):
    bar = 1e-12 if prec == G.GRAV_FP64 else 1e-5
    one, three = _plan(p, prec, 1), _plan(p, prec, 3)
    assert one.check() == "ok" and three.check() == "ok"
    gen = torch.Generator(device="cuda").manual_seed(p)
    rho = torch.randn(three.rho_shape, dtype=torch.float64, device="cuda", generator=gen)
    g3 = three.eval(rho)
    g1 = torch.stack([one.eval(rho[b].contiguous()) for b in range(3)])
    assert float((g3 - g1).norm() / g1.norm()) <= bar
    ref = one.direct(rho[0].contiguous())
    assert float((g1[0] - ref).norm() / ref.norm()) <= 2 * 0.55 ** p + bar
    r = torch.randn(three.out_shape, dtype=torch.float64, device="cuda", generator=gen)
    d3 = three.adjoint(r)
    d1 = torch.stack([one.adjoint(r[b].contiguous()) for b in range(3)])
    assert float((d3 - d1).norm() / d1.norm()) <= bar
    gap = abs(float((g3 * r).sum()) - float((rho * d3).sum())) / (float(g3.norm()) * float(r.norm()))
    assert gap <= bar
