"""More (source, model) pairs than one dimension of a launch holds (2^32 - 1
work-items): 70,000 scattered sources in 61,440 models, 34 GB of values, a
station above them.

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
