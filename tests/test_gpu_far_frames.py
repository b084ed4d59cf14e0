"""Points far from the origin for their extent, where floats are coarser than codes: the walks over codes lose
nothing there (against the oracle), and take about as long as for the same points at the origin."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dim", [2, 3, 6])
@pytest.mark.parametrize("far", [1e3, -2.0e4, 4.5e6, 3e7])
def test_far_points_match_the_oracle(dim, far):
    rng = np.random.default_rng([dim, int(abs(far))])
    pts = (rng.random((1200, dim)) * rng.choice([1.0, 300.0], dim) + far).astype(np.float32)
    lo, hi = pts.min(0), pts.max(0)
    q = np.concatenate([pts[::40], np.nextafter(pts[::50], np.float32(np.inf)), np.stack([lo, hi]),
                        lo + (hi - lo) * (3.0 * rng.random((60, dim)) - 1.0)]).astype(np.float32)
    t = ax.arborx_bvh_build(dev(pts))
    for k in (1, 6, 20):
        o_d2, o_ix = oracle.knn(pts, q, k, dim=dim)
        d2, ix = ax.arborx_query_knn(t, dev(q), k)
        assert np.array_equal(ix.cpu().numpy(), o_ix) and np.array_equal(d2.cpu().numpy(), o_d2), k
    ulp = float(np.spacing(np.float32(abs(far))))
    for r in (0.0, ulp, 0.3 * float((hi - lo).max()), 4.0):
        r = float(np.float32(r))
        o_off, o_idx = oracle.spatial(pts, q, r, dim=dim)
        off, idx = ax.arborx_query_spatial(t, dev(q), r)
        assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx), r
        s_off, _ = oracle.spatial(pts, pts, r, dim=dim)
        assert np.array_equal(ax.arborx_self_join_degree(t, r).cpu().numpy(), np.diff(s_off) - 1), r
    boxes = np.stack([q - np.float32(0.3), q + np.float32(0.3)], 1)  # these decode the boxes
    o_off, o_idx = oracle.intersects(pts, boxes, dim=dim)
    off, idx = ax.arborx_query_intersects(t, dev(boxes))
    assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx)


def seconds(call):
    call()
    best = np.inf
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 1e3)
    return best


def test_far_points_cost_what_near_ones_do():
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    near, q = (torch.rand((500_000, 3), generator=g, device="cuda") for _ in range(2))
    times = []
    for far in (0.0, 3.0e5):
        t = ax.arborx_bvh_build((near + far).contiguous())
        at = (q + far).contiguous()
        times.append([seconds(lambda: ax.arborx_query_knn(t, at, 8)),
                      seconds(lambda: ax.arborx_query_spatial_reduce(t, at, 0.017, ax.COUNT))])
    # with boxes and queries widened by the spacing of floats they took six times as long
    assert all(far < 2.5 * origin for origin, far in zip(*times)), times
