"""Queries outside a tree's frame: their excess past it enters the walks in codes (scaled where it is
above 16 bits).  Every result is compared with the oracle element by element."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def outside(dim, ratio, rng):
    """Queries `ratio` frames past one face, past several, past all, and across the border."""
    q = rng.random((48, dim), dtype=np.float32)
    side = rng.choice([-1, 0, 1], size=(48, dim))
    side[:dim] = np.eye(dim, dtype=side.dtype)
    side[dim:2 * dim] = -np.eye(dim, dtype=side.dtype)
    return np.where(side > 0, 1 + ratio * (0.5 + q), np.where(side < 0, -ratio * (0.5 + q), q)).astype(np.float32)


@pytest.mark.parametrize("dim", [2, 3, 6])
@pytest.mark.parametrize("ratio", [1e-4, 0.05, 0.49, 0.51, 1.0, 40.0, 3.0e4, 1e7])
def test_queries_outside_the_frame_match_the_oracle(dim, ratio):
    rng = np.random.default_rng([dim, int(ratio * 1e4)])
    for scale, shift in ((1.0, 0.0), (7.0, 1000.0)):
        pts = (rng.random((900, dim), dtype=np.float32) * np.float32(scale) + np.float32(shift)).astype(np.float32)
        q = (outside(dim, ratio, rng) * np.float32(scale) + np.float32(shift)).astype(np.float32)
        t = ax.arborx_bvh_build(dev(pts))
        dq = dev(q)
        for k in (1, 8, 33):
            o_d2, o_ix = oracle.knn(pts, q, k, dim=dim)
            d2, ix = ax.arborx_query_knn(t, dq, k)
            assert np.array_equal(ix.cpu().numpy(), o_ix) and np.array_equal(d2.cpu().numpy(), o_d2), (scale, k)
        near = float(np.sqrt(np.median(oracle.knn(pts, q, 8, dim=dim)[0][:, 7])))
        for r in (0.0, 0.9 * near, near, 1.3 * near, np.inf):
            r = float(np.float32(r))
            o_off, o_idx = oracle.spatial(pts, q, r, dim=dim)
            off, idx = ax.arborx_query_spatial(t, dq, r)
            assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx), (scale, r)
            c, _ = ax.arborx_query_spatial_reduce(t, dq, r, ax.COUNT)
            assert np.array_equal(c.cpu().numpy(), np.diff(o_off)), (scale, r)
