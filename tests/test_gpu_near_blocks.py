"""Near field of 4^3-cell leaves at the cell centres, both directions: the dense
matrices of plans whose blocks of leaves stay mostly empty (meshes of one leaf
or a row of them, many models) against the same models by parity, wide
transposed blocks on ragged meshes, meshes without a far field.

Bars: the forms differ in the order of sums, so rounding (1e-12 FP64, FP32
products 1e-6); without a far field the FMM is the direct sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")

PREC = pytest.mark.parametrize("prec, bar", [(G.GRAV_FP64, 1e-12), (G.GRAV_MIXED, 1e-6)], ids=["fp64", "mixed"])


def _plan(n, batch, comps, prec, points=None, p=6):
    return G.Plan(G.PlanSpec(n=n, h=1.0, voxel_centres=True, components=comps, p=p, leaf_size=64, points=points,
                             precision=prec, batch=batch))


def _randn(shape, seed):
    return torch.randn(shape, dtype=torch.float64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(seed))


def _gap(g, r, rho, d):
    return abs(float((g * r).sum()) - float((rho * d).sum())) / (float(g.norm()) * float(r.norm()))


@PREC
@pytest.mark.parametrize("comps", [1, 3, 4])
@pytest.mark.parametrize("n, batch", [((4, 4, 4), 1025), ((3, 4, 2), 1100), ((16, 4, 4), 2049), ((4, 4, 17), 700),
                                      ((7, 8, 3), 2100)])
def test_mostly_empty_blocks(n, batch, comps, prec, bar):
    pts = np.array([[1.2, 2.3, 0.7], [n[0] + 5.0, 1.0, 2.0]]) if n[0] > 4 else None
    many, one = _plan(n, batch, comps, prec, pts), _plan(n, 3, comps, prec, pts)
    assert many.check() == "ok"
    rho, r = _randn(many.rho_shape, 1), _randn(many.out_shape, 2)
    g, d = many.eval(rho), many.adjoint(r)
    for b in (0, batch // 2, batch - 3):
        ref = one.eval(rho[b:b + 3].contiguous())
        assert float((g[b:b + 3] - ref).norm() / ref.norm()) <= bar
        ref = one.adjoint(r[b:b + 3].contiguous())
        assert float((d[b:b + 3] - ref).norm() / ref.norm()) <= bar
    assert _gap(g, r, rho, d) <= bar


@pytest.mark.parametrize("comps", [1, 3, 4])
def test_wide_transposed_blocks(comps):
    """At least 16384 leaves over the models on a ragged mesh of 18 x 16 x 10."""
    n, batch = (70, 61, 37), 6
    many, one = _plan(n, batch, comps, G.GRAV_MIXED), _plan(n, 1, comps, G.GRAV_MIXED)
    rho, r = _randn(many.rho_shape, 1), _randn(many.out_shape, 2)
    d = many.adjoint(r)
    ref = torch.stack([one.adjoint(r[b].contiguous()) for b in range(batch)])
    assert float((d - ref).norm() / ref.norm()) <= 1e-6
    assert _gap(many.eval(rho), r, rho, d) <= 1e-6


@PREC
@pytest.mark.parametrize("comps", [1, 3, 4])
@pytest.mark.parametrize("n", [(4, 4, 4), (5, 8, 3), (8, 8, 8)])
def test_no_far_field(n, comps, prec, bar):
    plan = _plan(n, 2, comps, prec)
    assert plan.levels < 2
    rho, r = _randn(plan.rho_shape, 1), _randn(plan.out_shape, 2)
    g, d = plan.eval(rho), plan.adjoint(r)
    ref = plan.direct(rho)
    assert float((g - ref).norm()) <= bar * float(ref.norm())
    # the transpose, entry by entry: column j of the map is the field of cell j
    cell = torch.zeros_like(rho)
    flat = cell.reshape(2, -1)
    for j in {0, flat.shape[1] // 2, flat.shape[1] - 1}:
        flat.zero_()
        flat[:, j] = 1.0
        col = plan.direct(cell)
        got = d.reshape(2, -1)[:, j]
        scale = (col.abs() * r.abs()).sum((1, 2))
        assert bool(((got - (col * r).sum((1, 2))).abs() <= bar * scale).all())


@PREC
@pytest.mark.parametrize("comps", [1, 3, 4])
def test_one_cell(comps, prec, bar):
    """The only pair is the coincident one: zero up to the rounding of the
    parity sums, whose terms are the pair terms of the cell's mirror images (at
    most 1 in cell units)."""
    plan = _plan((1, 1, 1), 2, comps, prec)
    rho, r = _randn(plan.rho_shape, 1), _randn(plan.out_shape, 2)
    assert float(plan.eval(rho).abs().max()) <= bar * float(rho.abs().max())
    assert float(plan.adjoint(r).abs().max()) <= bar * float(r.abs().sum((1, 2)).max())
