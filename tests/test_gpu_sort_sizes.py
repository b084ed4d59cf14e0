"""The sort at the sizes where its method changes: one tile, merges of runs (whole and ragged), and
radix tiles of 4, 8 and 16 keys per thread; against numpy's stable sort."""
import numpy as np
import pytest

import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [2, 63, 65, 1023, 1024, 1025, 8191, 8193, 20_000, 65_535, 65_536, 65_537, 300_001,
                               524_288, 524_289, 2_000_000, 2_000_001])
@pytest.mark.parametrize("bits,lo,hi", [(64, 0, 63), (64, 0, 64), (64, 5, 37), (32, 0, 24), (32, 0, 32), (32, 3, 27)])
def test_stable_at_every_size(n, bits, lo, hi):
    g = np.random.default_rng([n, bits, lo])
    dt = np.uint64 if bits == 64 else np.uint32
    width = hi - lo
    mask = dt((1 << width) - 1)
    for few in (False, True):
        k = g.integers(0, 2 ** bits, n, dtype=dt)
        if few:  # many equal keys, the largest among them
            k = np.where(k % dt(5) == 0, ~dt(0), k % dt(3)).astype(dt)
        v = g.permutation(n).astype(np.int32)
        dk = torch.from_numpy(k.view(np.int64 if bits == 64 else np.int32).copy()).cuda()
        dv = torch.from_numpy(v).cuda()
        ax.arborx_debug_radix_sort(dk, dv, lo, hi)
        order = np.argsort((k >> dt(lo)) & mask, kind="stable")
        assert np.array_equal(dv.cpu().numpy(), v[order])
        assert np.array_equal(dk.cpu().numpy().view(dt), k[order])


@pytest.mark.parametrize("n", [700, 5000, 9000])
def test_build_from_either_buffer(n):
    """Trees whose sort ends in the first or the second buffer: codes kept for kNN seeds included."""
    import oracle
    g = np.random.default_rng(n)
    pts, q = g.random((n, 3), dtype=np.float32), g.random((200, 3), dtype=np.float32)
    t = ax.arborx_bvh_build(torch.from_numpy(pts).cuda())
    torch.cuda.synchronize()
    other = ax.arborx_bvh_build(torch.from_numpy(pts[::-1].copy()).cuda())  # takes the blocks the first build freed
    d2, ix = ax.arborx_query_knn(t, torch.from_numpy(q).cuda(), 5)
    o_d2, o_ix = oracle.knn(pts, q, 5)
    assert np.array_equal(ix.cpu().numpy(), o_ix) and np.array_equal(d2.cpu().numpy(), o_d2)
    assert other.n == n
