"""L2P of leaves that hold many points, whose points are cut into runs: run
ends on and off whole steps of 64 (point, model) pairs, one and several groups
of models, single points in other leaves.  Many leaves of a single model, up to
16 of whose runs share a workgroup.

Bar: a point's field does not depend on the other points of its plan, so every
field equals that of the same point in plans of few points (the same tree, no
leaf in more than one run) to FP64 rounding, 1e-12."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
G = pytest.importorskip("paper_1107_5951_amd")


@pytest.mark.parametrize("batch", [1, 3, 8, 9])
@pytest.mark.parametrize("npts", [63, 64, 65, 127, 128, 1000])
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


@pytest.mark.parametrize("p, leaves, per, batch", [(10, 512, 1, 1), (10, 1025, 9, 1), (10, 2049, 70, 1), (3, 4097, 20, 1),
                                                   (10, 8191, 3, 1), (16, 8192, 11, 1), (10, 4096, 5, 2), (16, 4096, 2, 3),
                                                   (4, 8192, 3, 8), (16, 2049, 2, 9), (10, 4096, 1, 17)])
def test_runs_per_workgroup(p, leaves, per, batch):
    """Plans of no more than 256 leaves take a workgroup per run."""
    n = np.array([128, 64, 64])
    rng = np.random.default_rng(leaves)
    ids = rng.permutation(n.prod() // 64)[:leaves]
    corner = 4.0 * np.stack([ids % 32, ids // 32 % 16, ids // 512], axis=1)
    pts = np.repeat(corner, per, axis=0)
    pts = pts + rng.uniform(0.1, 3.9, size=pts.shape)

    def plan(pts, batch):
        return G.Plan(G.PlanSpec(n=tuple(int(v) for v in n), h=1.0, voxel_centres=False, components=3, p=p, leaf_size=64,
                                 points=pts, precision=G.GRAV_FP64, batch=batch))

    whole = plan(pts, batch)
    assert whole.n_target_leaves == leaves
    rho = torch.randn(whole.rho_shape, dtype=torch.float64, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(leaves))
    g = whole.eval(rho).reshape(batch, -1, 3)
    for at in (0, leaves // 2, leaves - 256):
        few = plan(pts[at * per:(at + 256) * per], 1)
        for b in (0, batch - 1):
            ref = few.eval(rho.reshape(batch, -1)[b].reshape(few.rho_shape)).reshape(-1, 3)
            assert float((g[b, at * per:(at + 256) * per] - ref).norm() / ref.norm()) <= 1e-12
