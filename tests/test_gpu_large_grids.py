"""More (source, model) pairs than a launch of one dimension holds: past 2^32
work-items the runtime starts the remainder of the count alone and reports no
error.  70,000 scattered sources in 61,440 models, 34 GB of values, a station
above them; as many (station, model) pairs, whose residual weights and fields
are written by a work-item each.

Bar: every model holds the first one's values times its own factor, a power of
two, so every field is that multiple of the first's exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


def test_scattered_masses_of_many_models():
    n, batch = 70000, 61440
    assert n * batch > 1 << 32
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 90 GB of free device memory")
    src = np.random.default_rng(1).uniform(0.0, 1.0, size=(n, 3)) * np.array([8.0, 8.0, 8.0])
    plan = G.Plan(G.PlanSpec(n=(8, 8, 8), h=1.0, points=np.array([[4.1, 3.9, 9.5]]), components=1, p=1, leaf_size=512,
                             precision=G.GRAV_FP64, batch=batch, sources=src))
    assert plan.levels < 2
    gen = torch.Generator(device="cuda").manual_seed(1)
    first = torch.rand(n, dtype=torch.float64, device="cuda", generator=gen)
    factor = torch.exp2((torch.arange(batch, device="cuda") % 11).double())
    rho = factor[:, None] * first[None, :]
    g = plan.eval(rho)[:, 0, 0]
    assert float(g[0]) > 0.0 and bool((g == g[0] * factor).all())
    del rho, plan
    torch.cuda.empty_cache()


def test_stations_of_many_models():
    n, batch = 70000, 61440
    assert n * batch > 1 << 32
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GB of free device memory")
    pts = np.random.default_rng(3).uniform(0.0, 2.0, size=(n, 3)) * np.array([8.0, 8.0, 1.0]) + np.array([0.0, 0.0, 3.0])
    plan = G.Plan(G.PlanSpec(n=(16, 16, 2), h=1.0, points=pts, components=1, p=2, leaf_size=1, precision=G.GRAV_FP64,
                             batch=batch))
    gen = torch.Generator(device="cuda").manual_seed(2)
    factor = torch.exp2((torch.arange(batch, device="cuda") % 11).double())
    for call, shape in ((plan.eval, plan.rho_shape), (plan.adjoint, plan.out_shape)):
        x = torch.empty(shape, dtype=torch.float64, device="cuda").reshape(batch, -1)
        first = torch.rand(x.shape[1], dtype=torch.float64, device="cuda", generator=gen)
        torch.mul(first[None, :], factor[:, None], out=x)
        y = call(x.reshape(shape)).reshape(batch, -1)
        del x
        assert bool((y[0] != 0.0).all())
        y /= factor[:, None]
        assert bool((y.amax(0) == y[0]).all() and (y.amin(0) == y[0]).all())
        del y
    del plan
    torch.cuda.empty_cache()
