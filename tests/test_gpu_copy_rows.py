"""Copy of the stash rows through LDS and of the offsets: row lengths around the stash's, the last
wavefront, tiles of the scan."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dim", [2, 3, 6])
@pytest.mark.parametrize("m", [1, 63, 65, 257, 4095, 4097, 8200])
def test_rows_of_every_length(dim, m):
    # points on a line at distance 1: a query at x with radius r meets an exact count of them
    n = 80
    pts = np.zeros((n, dim), dtype=np.float32)
    pts[:, 0] = np.arange(n, dtype=np.float32)
    rng = np.random.default_rng([dim, m])
    pts = pts[rng.permutation(n)]
    q = np.zeros((m, dim), dtype=np.float32)
    for r in (0.4, 7.6, 8.1, 15.7, 16.1, 40.0):  # rows of 0 .. 2 r + 1, fewer past the ends
        q[:, 0] = rng.integers(-45, n + 45, m).astype(np.float32)
        t = ax.arborx_bvh_build(dev(pts))
        o_off, o_idx = oracle.spatial(pts, q, r, dim=dim)
        for ordered in (True, False):
            off, idx = ax.arborx_query_spatial(t, dev(q), r, ordered=ordered)
            off, idx = off.cpu().numpy(), idx.cpu().numpy()
            assert np.array_equal(off, o_off), (r, ordered)
            if not ordered:  # rows hold the same indices in some order
                row = np.repeat(np.arange(m), np.diff(off))
                idx = idx[np.lexsort((idx, row))]
            assert np.array_equal(idx, o_idx), (r, ordered)
