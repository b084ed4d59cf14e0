"""DBSCAN where a wavefront's points belong to many clusters: their smallest indices (against the oracle), and
what it costs when every point is a cluster of its own."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# sizes of clusters that are neighbours in sorted order: all single, pairs, fewer and more a wavefront than are
# taken in turns (4), one large one between single points
@pytest.mark.parametrize("sizes", [[1], [2], [1, 2, 3], [13], [16], [21], [32, 32, 1], [40, 1, 1, 1], [200, 1]])
@pytest.mark.parametrize("min_pts", [1, 2, 5])
def test_smallest_index_of_each_cluster(sizes, min_pts):
    rng = np.random.default_rng([min_pts, *sizes])
    size = np.resize(sizes, 400)
    at = np.repeat(np.arange(400), size)
    pts = np.stack([10.0 * at, 0.001 * rng.random(len(at)), np.zeros(len(at))], 1).astype(np.float32)
    pts = pts[rng.permutation(len(pts))][:1700]
    t = ax.arborx_bvh_build(dev(pts))
    labels = ax.arborx_dbscan(t, dev(pts), 0.5, min_pts)
    assert np.array_equal(labels.cpu().numpy(), oracle.dbscan(pts, 0.5, min_pts))


def test_single_points_cost_no_turn_each():
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    pts = torch.rand((4000000, 3), generator=g, device="cuda")
    t = ax.arborx_bvh_build(pts)

    def seconds(min_pts):
        best = np.inf
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ax.arborx_dbscan(t, pts, 1e-5, min_pts)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) / 1e3)
        return best

    # without a core point the smallest indices are left out: one read and one atomic a point, not 64 turns (twice the time)
    clusters, noise = seconds(1), seconds(9)
    assert clusters < 1.5 * noise, (clusters, noise)
