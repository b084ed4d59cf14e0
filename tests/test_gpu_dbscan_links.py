"""DBSCAN's links over sorted positions: labels stay the smallest core value index whatever order the
values come in; wavefront edges; rows longer than the queue of a thread; several clusters a wavefront."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def check(pts, eps, min_pts):
    pts = np.ascontiguousarray(pts, dtype=np.float32)
    got = ax.BVH(torch.from_numpy(pts).cuda()).dbscan(eps, min_pts).cpu().numpy()
    assert np.array_equal(got, oracle.dbscan(pts, eps, min_pts, dim=pts.shape[1])), (len(pts), eps, min_pts)


@pytest.mark.parametrize("order", ["random", "sorted", "reversed"])
@pytest.mark.parametrize("dim", [2, 3, 6])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 257, 3000])
def test_labels_do_not_depend_on_the_input_order(order, dim, n):
    rng = np.random.default_rng([dim, n])
    pts = rng.random((n, dim), dtype=np.float32)
    pts[:, 0] = np.float32(0.5) * np.round(pts[:, 0] * 8)  # sheets: several clusters
    by = np.lexsort(pts.T)
    pts = pts if order == "random" else pts[by if order == "sorted" else by[::-1]]
    h = float(n) ** (-1.0 / max(1, dim - 1))
    for eps, min_pts in ((0.7 * h, 2), (1.5 * h, 5), (3.0 * h, 1), (4.0, 3)):
        check(pts, float(np.float32(eps)), min_pts)


@pytest.mark.parametrize("tuning", [dict(block=256, stack=64), dict(block=64, stack=1)])
def test_queue_beside_deep_and_shallow_stacks(tuning):
    rng = np.random.default_rng(5)
    pts = rng.random((2500, 3), dtype=np.float32)
    ax.arborx_set_tuning(node_format=1, queries_per_thread=1, **tuning)
    try:
        check(pts, 0.1, 8)
        t = ax.arborx_bvh_build(torch.from_numpy(pts).cuda())
        off, idx, _ = ax.arborx_query_spatial_with_distances(t, torch.from_numpy(pts).cuda(), 0.1)
        o_off, o_idx = oracle.spatial(pts, pts, 0.1)
        assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx)
    finally:
        ax.arborx_reset_tuning()
