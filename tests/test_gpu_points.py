"""L2P at user points and its transpose: leaves with one point and with more
than a wave or a chunk of 16, several leaves per workgroup, single models and
more than a group of eight, all cell centres by points (leaf edges without
lattice matrices), no far field.

Bars: the FMM against the direct sum within 2 x 0.55^p (one-box separation
converges like 0.4 .. 0.5 per order) and FP64 rounding; the transpose and the
batch against single models to rounding, 1e-12."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


def _points(kind):
    rng = np.random.default_rng(7)
    if kind == "dense":  # 150 and 17 points in two leaves
        return np.concatenate([rng.uniform(0.1, 2.9, size=(150, 3)), rng.uniform(0.1, 2.9, size=(17, 3)) + [6, 3, 9]])
    return rng.uniform(-2.0, 20.0, size=(200, 3))  # about one per leaf


@pytest.mark.parametrize("kind", ["dense", "few", "centres", "one leaf"])
@pytest.mark.parametrize("p", [1, 7, 12, 16])
def test_points(p, kind):
    leaf = {"dense": 27, "few": 8, "centres": 216, "one leaf": 512}[kind]
    n = (7, 6, 5) if kind == "one leaf" else (19, 16, 13)

    def plan(batch):
        return G.Plan(G.PlanSpec(n=n, h=1.0, voxel_centres=kind in ("centres", "one leaf"), components=4, p=p,
                                 leaf_size=leaf, points=_points(kind), precision=G.GRAV_FP64, batch=batch))

    one, many = plan(1), plan(9)
    gen = torch.Generator(device="cuda").manual_seed(p)
    rho = torch.randn(many.rho_shape, dtype=torch.float64, device="cuda", generator=gen)
    g = many.eval(rho)
    ref = torch.stack([one.eval(rho[b].contiguous()) for b in range(9)])
    assert float((g - ref).norm() / ref.norm()) <= 1e-12
    direct = one.direct(rho[0].contiguous())
    assert float((ref[0] - direct).norm() / direct.norm()) <= 2 * 0.55 ** p + 1e-12
    r = torch.randn(many.out_shape, dtype=torch.float64, device="cuda", generator=gen)
    d = many.adjoint(r)
    ref = torch.stack([one.adjoint(r[b].contiguous()) for b in range(9)])
    assert float((d - ref).norm() / ref.norm()) <= 1e-12
    gap = abs(float((g * r).sum()) - float((rho * d).sum())) / (float(g.norm()) * float(r.norm()))
    assert gap <= 1e-12
