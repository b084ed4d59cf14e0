"""Launches of few queries use small workgroups: results around the sizes where the workgroup changes."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dim", [2, 3, 6])
@pytest.mark.parametrize("m", [1, 7, 9, 4095, 8177, 16353, 32705, 32769])
def test_few_queries_match_the_oracle(dim, m):
    rng = np.random.default_rng([dim, m])
    pts = rng.random((700, dim), dtype=np.float32)
    q = (rng.random((m, dim), dtype=np.float32) * np.float32(1.2) - np.float32(0.1)).astype(np.float32)
    r = float(np.float32({2: 0.11, 3: 0.2, 6: 0.45}[dim]))  # some rows longer than the stash
    t, dq = ax.arborx_bvh_build(dev(pts)), dev(q)
    o_off, o_idx = oracle.spatial(pts, q, r, dim=dim)
    off, idx = ax.arborx_query_spatial(t, dq, r)
    assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx)
    off, idx, _ = ax.arborx_query_spatial_with_distances(t, dq, r)
    assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx)
    o_c, o_s = oracle.reduce(pts, q, r, dim=dim)
    c, s = ax.arborx_query_spatial_reduce(t, dq, r, ax.COUNT_SUMDIST)
    assert np.array_equal(c.cpu().numpy(), o_c) and np.array_equal(s.cpu().numpy(), o_s)
    few = ax.arborx_query_spatial_count_up_to(t, dq, r, 3)
    assert np.array_equal(few.cpu().numpy(), np.minimum(o_c, 3))
    for k in (1, 10):
        o_d2, o_ix = oracle.knn(pts, q, k, dim=dim)
        d2, ix = ax.arborx_query_knn(t, dq, k)
        assert np.array_equal(ix.cpu().numpy(), o_ix) and np.array_equal(d2.cpu().numpy(), o_d2)
