"""Points much closer together than the codes of their tree's frame: one stray point far away, or half of the
points in a clump.  Walks over codes would meet every point of the crowd there, thousands of times the
work; the results are compared with the oracle, and the time with that of the same number of even points."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MOST = 40.0  # times the even set's time; a walk that meets the whole crowd takes hundreds of times as long


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def sets(dim, n, rng):
    even = rng.random((n, dim), dtype=np.float32)
    stray = even.copy()
    stray[n // 3] = 1.0e5
    clump = even.copy()
    clump[: n // 2] = np.float32(0.5) + (even[: n // 2] - np.float32(0.5)) * np.float32(2e-5)
    return even, {"stray": stray, "clump": clump}


def seconds(call):
    call()
    best = np.inf
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 1e3)
    return best


@pytest.mark.parametrize("dim", [2, 3])
def test_nearest_and_small_balls_among_crowded_points(dim):
    n = 200_000
    even, crowded = sets(dim, n, np.random.default_rng(dim))
    cut = [0, n // 2, n]
    bo, bt = dev(np.array(cut, np.int64)), dev(np.arange(2, dtype=np.int32))
    r = float(np.float32(0.3 * n ** (-1.0 / dim)))
    br = dev(np.full(2, r, np.float32))

    def calls(pts):
        d = dev(pts)
        tree, forest = ax.arborx_bvh_build(d), ax.arborx_forest_build(d, cut)
        # among crowded points, balls of a hundredth of the clump's width: few matches, as in the even set
        small = r if pts is even else 2e-7
        return [lambda: ax.arborx_query_knn(tree, d, 6), lambda: ax.arborx_forest_query_knn(forest, d, bo, bt, 6),
                lambda: ax.arborx_query_spatial_reduce(tree, d, small, ax.COUNT)]

    base = [seconds(c) for c in calls(even)]
    few = np.random.default_rng(1).integers(0, n, 200)
    for name, pts in crowded.items():
        for call, plain in zip(calls(pts), base):
            assert seconds(call) < MOST * plain, name
        tree = ax.arborx_bvh_build(dev(pts))
        q = np.ascontiguousarray(pts[few])
        o_d2, o_ix = oracle.knn(pts, q, 6, dim=dim)
        d2, ix = ax.arborx_query_knn(tree, dev(q), 6)
        assert np.array_equal(ix.cpu().numpy(), o_ix) and np.array_equal(d2.cpu().numpy(), o_d2), name
        for radius in (1e-6, 1e-4, r):
            radius = float(np.float32(radius))
            off, idx = ax.arborx_query_spatial(tree, dev(q), radius)
            o_off, o_idx = oracle.spatial(pts, q, radius, dim=dim)
            assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx), (name, radius)


@pytest.mark.parametrize("dim", [2, 3, 6])
@pytest.mark.parametrize("n", [9, 300, 5000])  # a crowd inside a chunk of the build, and over several
def test_crowds_inside_and_across_the_parts_of_a_build(dim, n):
    rng = np.random.default_rng([dim, n])
    pts = np.ascontiguousarray(np.concatenate([rng.random((20, dim), dtype=np.float32),
                                               np.float32(0.4) + rng.random((n, dim), dtype=np.float32) * np.float32(3e-5)]))
    q = np.ascontiguousarray(pts[rng.integers(0, len(pts), 60)])
    for build in (0, 1):
        ax.arborx_set_tuning(build=build, node_format=1)
        try:
            tree = ax.arborx_bvh_build(dev(pts))
            d2, ix = ax.arborx_query_knn(tree, dev(q), 7)
            c, _ = ax.arborx_query_spatial_reduce(tree, dev(q), 1e-5, ax.COUNT)
            deg = ax.arborx_self_join_degree(tree, 1e-5)
        finally:
            ax.arborx_reset_tuning()
        o_d2, o_ix = oracle.knn(pts, q, 7, dim=dim)
        assert np.array_equal(ix.cpu().numpy(), o_ix) and np.array_equal(d2.cpu().numpy(), o_d2)
        o_off, _ = oracle.spatial(pts, q, float(np.float32(1e-5)), dim=dim)
        assert np.array_equal(c.cpu().numpy(), np.diff(o_off))
        s_off, _ = oracle.spatial(pts, pts, float(np.float32(1e-5)), dim=dim)
        assert np.array_equal(deg.cpu().numpy(), np.diff(s_off) - 1)
