"""Lattice near field of leaves of 1 to 27 cells at 8192 tiles or more, where a
wave has a tile of its own, against the same models alone, where four waves
share one; the transpose against both.

Bars: the forms differ in the order of sums, so rounding (1e-12 FP64, FP32
products 1e-6; the FP32 M2L's dot product 1e-5)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


def _randn(shape, seed):
    return torch.randn(shape, dtype=torch.float64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(seed))


@pytest.mark.parametrize("n, leaf, comps, batch, prec", [
    ((64, 62, 64), 27, 3, 13, G.GRAV_MIXED),
    ((64, 62, 64), 27, 3, 9, G.GRAV_FP64),
    ((64, 62, 64), 27, 1, 26, G.GRAV_MIXED),
    ((64, 63, 64), 8, 3, 8, G.GRAV_MIXED),
    ((64, 63, 64), 8, 4, 4, G.GRAV_FP64),
    ((48, 48, 47), 1, 4, 3, G.GRAV_MIXED),
    ((48, 48, 47), 1, 3, 2, G.GRAV_FP64),
])
def test_tile_per_wave(n, leaf, comps, batch, prec):
    bar, gap_bar = (1e-12, 1e-12) if prec == G.GRAV_FP64 else (1e-6, 1e-5)

    def plan(b):
        return G.Plan(G.PlanSpec(n=n, h=1.0, voxel_centres=True, components=comps, p=4, leaf_size=leaf, precision=prec,
                                 batch=b))

    many, one = plan(batch), plan(1)
    edge = round(leaf ** (1 / 3))
    assert many.leaf_cells == edge
    rows = comps * -(-leaf // 16)
    tiles = -(-int(np.prod([-(-k // edge) for k in n])) * batch // 32) * -(-rows // (2 if prec == G.GRAV_FP64 else 4))
    assert tiles >= 8192 and tiles // batch < 8192
    rho, r = _randn(many.rho_shape, 1), _randn(many.out_shape, 2)
    g, d = many.eval(rho), many.adjoint(r)
    for b in (0, batch - 1):
        ref = one.eval(rho[b].contiguous().reshape(one.rho_shape)).reshape(g[b].shape)
        assert float((g[b] - ref).norm() / ref.norm()) <= bar
        ref = one.adjoint(r[b].contiguous().reshape(one.out_shape)).reshape(d[b].shape)
        assert float((d[b] - ref).norm() / ref.norm()) <= bar
    assert abs(float((g * r).sum()) - float((rho * d).sum())) / (float(g.norm()) * float(r.norm())) <= gap_bar
