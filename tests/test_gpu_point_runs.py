"""L2P of leaves that hold many points, whose points are cut into runs: run
ends on and off whole steps of 64 (point, model) pairs, one and several groups
of models, single points in other leaves.

Bar: a point's field does not depend on the other points of its plan, so every
field equals that of the same point in plans of few points (the same tree, no
leaf in more than one run) to FP64 rounding, 1e-12."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


@pytest.mark.parametrize("batch", [1, 3, 8, 9])
@pytest.mark.parametrize("npts", [63, 64, 65, 1000])
def test_point_runs(npts, batch):
    rng = np.random.default_rng(npts)
    frame = np.array([[-3.0, -3.0, -3.0], [30.0, 30.0, 30.0]])  # in every plan: one root box
    pts = rng.uniform(0.1, 3.9, size=(npts, 3)) + [12.0, 8.0, 20.0]  # one leaf, away from the mesh

    def plan(p):
        return G.Plan(G.PlanSpec(n=(16, 16, 16), h=1.0, voxel_centres=False, components=3, p=7, leaf_size=64,
                                 points=np.concatenate([p, frame]), precision=G.GRAV_FP64, batch=batch))

    whole = plan(pts)
    assert whole.n_target_leaves == 3
    rho = torch.randn(whole.rho_shape, dtype=torch.float64, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(npts))
    g = whole.eval(rho)
    few = 7 if batch > 1 else 63  # a run is at most 64 / min(batch, 8) points here
    for at in range(0, npts, few):
        ref = plan(pts[at:at + few]).eval(rho)[:, :-2]
        assert float((g[:, at:at + few][:, :ref.shape[1]] - ref).norm() / ref.norm()) <= 1e-12
