"""Rows sorted by a wavefront (up to 256 entries, one, two or four a lane) or a workgroup (up to 1024),
in every order the searches return: by index, by index with values, by value."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENGTHS = [17, 33, 63, 64, 65, 127, 128, 129, 200, 255, 256, 257, 500, 1023, 1024, 1025, 1300]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dim", [2, 3, 6])
def test_rows_around_every_length(dim):
    n = 1400
    rng = np.random.default_rng(dim)
    pts = np.zeros((n, dim), dtype=np.float32)
    pts[:, 0] = rng.permutation(n).astype(np.float32)
    for want in LENGTHS:
        q = np.zeros((40, dim), dtype=np.float32)
        q[:, 0] = np.arange(40) - 20.0  # up to `want` points within reach, one fewer a step past the end
        r = float(want) - 0.5
        t = ax.arborx_bvh_build(dev(pts))
        o_off, o_idx = oracle.spatial(pts, q, r, dim=dim)
        assert want in np.diff(o_off)
        off, idx, d2 = ax.arborx_query_spatial_with_distances(t, dev(q), r)
        assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx), want
        row = np.repeat(np.arange(40), np.diff(o_off))
        assert np.array_equal(d2.cpu().numpy(), (pts[o_idx, 0] - q[row, 0]) ** 2), want
        off, idx = ax.arborx_query_spatial(t, dev(q), r)
        assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx), want


def test_rays_in_the_order_met():
    n = 1400
    rng = np.random.default_rng(7)
    lo = np.zeros((n, 3), dtype=np.float32)
    lo[:, 0] = rng.permutation(n) // 2  # pairs entered at once: ties go by index
    b = np.stack([lo, lo + np.float32(0.5)], axis=1)
    start = np.concatenate([n // 2 - (np.array(LENGTHS) + 1) // 2, np.arange(650, 700)]).astype(np.float32)
    rays = np.zeros((len(start), 2, 3), dtype=np.float32)
    rays[:, 0, 0] = start - np.float32(0.25)
    rays[:, 0, 1:] = 0.25
    rays[:, 1, 0] = 0.5
    t = ax.arborx_bvh_build(dev(b), ax.BOXES)
    off, idx, te = ax.arborx_query_ray_ordered_intersect(t, dev(rays))
    o_off, o_idx, o_t = oracle.ray_ordered_intersect(b, rays, dim=3, kind=oracle.BOXES)
    assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx)
    assert np.array_equal(te.cpu().numpy(), o_t)
