"""Device blocks kept between calls: results stay exact while several threads, each on its own
stream, build, query and destroy trees at once (a block handed over too early would be written by
two of them), and the kept memory goes back to the device when a caller installs an allocator."""
import gc
import threading

import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax
from paper_2507_23700_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def work(seed, n, out, rounds):
    stream = torch.cuda.Stream()
    g = np.random.default_rng(seed)
    data, q = inputs.cube(n, 3, g), inputs.cube(n // 2, 3, g)
    r = float(inputs.radius_cube(n, 12.0))
    with torch.cuda.stream(stream):
        d, dq = torch.from_numpy(data).cuda(), torch.from_numpy(q).cuda()
        got = []
        for _ in range(rounds):
            t = ax.arborx_bvh_build(d)
            off, idx = ax.arborx_query_spatial(t, dq, r)
            d2, near = ax.arborx_query_knn(t, dq, 4)
            got.append((off, idx, d2, near))
            del t
    stream.synchronize()
    out[seed] = (data, q, r, [[x.cpu().numpy() for x in v] for v in got])


@pytest.mark.parametrize("threads", [1, 3])
def test_kept_blocks_between_streams(threads):
    out = {}
    # sizes near each other, so that blocks of one thread fit the others
    ts = [threading.Thread(target=work, args=(s, 6000 + 37 * s, out, 4)) for s in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert len(out) == threads
    for data, q, r, got in out.values():
        o_off, o_idx = oracle.spatial(data, q, r)
        o_d2, o_near = oracle.knn(data, q, 4)
        for off, idx, d2, near in got:
            assert np.array_equal(off, o_off) and np.array_equal(idx, o_idx)
            assert np.array_equal(d2, o_d2) and np.array_equal(near, o_near)


def test_tree_used_on_two_streams_is_released_after_both():
    g = np.random.default_rng(9)
    data, q = inputs.cube(30_000, 3, g), inputs.cube(20_000, 3, g)
    o_d2, o_near = oracle.knn(data, q, 10)
    d, dq = torch.from_numpy(data).cuda(), torch.from_numpy(q).cuda()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got = []
    for _ in range(4):
        t = ax.arborx_bvh_build(d)
        got.append(ax.arborx_query_knn(t, dq, 10))
        with torch.cuda.stream(side):
            got.append(ax.arborx_query_knn(t, dq, 10, stream=side))
        del t  # the next build may only take this memory after the side stream's walk
    side.synchronize()
    torch.cuda.synchronize()
    for d2, near in got:
        assert np.array_equal(d2.cpu().numpy(), o_d2) and np.array_equal(near.cpu().numpy(), o_near)


def test_kept_memory_is_given_back():
    d = torch.rand((4_000_000, 3), device="cuda")
    t = ax.arborx_bvh_build(d)
    ax.arborx_query_knn(t, d[:1000], 4)
    del t
    gc.collect()
    torch.cuda.synchronize()
    kept = torch.cuda.mem_get_info()[0]
    ax.use_torch_allocator()  # needs nothing of the library's own: all of it goes back
    try:
        assert torch.cuda.mem_get_info()[0] >= kept + 4_000_000 * 64  # the nodes at least
    finally:
        ax.arborx_set_allocator()
