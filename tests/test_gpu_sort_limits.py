"""The sort at the numbers of keys where its tiles change, and the allocation-free nearest search at its most
queries, whose workspace has to hold the tiles of every number up to there."""
import numpy as np
import pytest

import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LIMITS = [3 << 18, 31 << 16]


@pytest.mark.parametrize("n", [x + d for x in LIMITS for d in (-1, 0, 1)])
@pytest.mark.parametrize("bits,lo,hi", [(64, 0, 63), (32, 0, 24)])
def test_stable_at_the_limits(n, bits, lo, hi):
    g = np.random.default_rng([n, bits])
    dt = np.uint64 if bits == 64 else np.uint32
    k = g.integers(0, 2 ** bits, n, dtype=dt)
    k[::7] = dt(12345)
    v = g.permutation(n).astype(np.int32)
    dk = torch.from_numpy(k.view(np.int64 if bits == 64 else np.int32).copy()).cuda()
    dv = torch.from_numpy(v).cuda()
    ax.arborx_debug_radix_sort(dk, dv, lo, hi)
    order = np.argsort((k >> dt(lo)) & dt((1 << (hi - lo)) - 1), kind="stable")
    assert np.array_equal(dv.cpu().numpy(), v[order]) and np.array_equal(dk.cpu().numpy().view(dt), k[order])


@pytest.mark.parametrize("m", [LIMITS[1] - 1, LIMITS[1], ax.NOALLOC_MAX_QUERIES])
def test_allocation_free_search_takes_its_most_queries(m):
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    pts = torch.rand((2000, 3), generator=g, device="cuda")
    q = torch.rand((m, 3), generator=g, device="cuda")
    t = ax.arborx_bvh_build(pts)
    d2, ix = ax.arborx_query_knn(t, q, 2)
    got_d2, got_ix = ax.arborx_query_knn_noalloc(t, q, 2)
    assert torch.equal(ix, got_ix) and torch.equal(d2, got_d2)
