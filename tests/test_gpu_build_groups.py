"""The chunked climb at the sizes where its levels change (one chunk, one group of chunks, several
groups), against the single-pass climb node by node, and its quantized nodes by what walks over them
find."""
import numpy as np
import pytest

import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def points(n, dim, kind, seed):
    g = np.random.default_rng([n, dim, seed])
    if kind == "uniform":
        return g.random((n, dim), dtype=np.float32)
    if kind == "equal":  # split keys from positions alone
        return np.full((n, dim), 0.5, np.float32)
    a = g.random((n, dim), dtype=np.float32) ** 6  # most values near one corner, long chains of levels
    a[: n // 3] = a[g.integers(0, n, n // 3)]
    return np.ascontiguousarray(a)


@pytest.fixture(autouse=True)
def _defaults():
    yield
    ax.arborx_reset_tuning()


@pytest.mark.parametrize("kind", ["uniform", "equal", "clumped"])
@pytest.mark.parametrize("dim,n", [(3, 1024), (3, 1025), (3, 2049), (3, 131_072), (3, 131_073), (3, 300_001),
                                   (2, 140_000), (6, 512), (6, 513), (6, 66_000)])
def test_same_tree_as_the_single_pass(dim, n, kind):
    d = torch.from_numpy(points(n, dim, kind, 1)).cuda()
    t = ax.arborx_bvh_build(d)
    a, ia = ax.arborx_debug_tree_nodes(t), ax.arborx_bvh_info(t)
    q = d[:: max(1, n // 700)].contiguous()
    r = 0.0 if kind == "equal" else 0.02 if dim < 6 else 0.1
    count = ax.arborx_query_spatial_reduce(t, q, r, ax.COUNT)[0]
    d2, ix = ax.arborx_query_knn(t, q, 5)
    ax.arborx_set_tuning(build=1, node_format=0)
    s = ax.arborx_bvh_build(d)
    b, ib = ax.arborx_debug_tree_nodes(s), ax.arborx_bvh_info(s)
    assert ia == ib and a[3] == b[3]
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)
    assert torch.equal(count, ax.arborx_query_spatial_reduce(s, q, r, ax.COUNT)[0])
    e2, jx = ax.arborx_query_knn(s, q, 5)
    assert torch.equal(ix, jx) and torch.equal(d2, e2)


def test_forest_across_groups():
    """Trees that end inside chunks, at their borders, and span groups of chunks, some of one value."""
    g = np.random.default_rng(3)
    sizes = [1, 1023, 1, 1024, 140_000, 1, 3, 2500, 0, 1, 60_000]
    vals = torch.from_numpy(g.random((sum(sizes), 3), dtype=np.float32)).cuda()
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    f = ax.arborx_forest_build(vals, off)
    roots = f.info()["roots"]
    q = torch.from_numpy(g.random((300 * len(sizes), 3), dtype=np.float32)).cuda()
    boff = torch.arange(len(sizes) + 1, dtype=torch.int64, device="cuda") * 300
    tree = torch.arange(len(sizes), dtype=torch.int32, device="cuda")
    rad = torch.full((len(sizes),), 0.05, device="cuda")
    c, _ = f.reduce(q, boff, tree, rad, ax.COUNT)
    d2, ix = f.knn(q, boff, tree, 4)
    for t, n in enumerate(sizes):
        assert (roots[t] >= 0) == (n > 0)
        one = ax.arborx_bvh_build(vals[off[t]:off[t + 1]].contiguous())
        sl = slice(300 * t, 300 * (t + 1))
        assert torch.equal(c[sl], ax.arborx_query_spatial_reduce(one, q[sl].contiguous(), 0.05, ax.COUNT)[0])
        e2, jx = ax.arborx_query_knn(one, q[sl].contiguous(), 4)
        assert torch.equal(ix[sl], jx) and torch.equal(d2[sl], e2)
