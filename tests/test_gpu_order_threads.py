"""Concurrent queries on one tree with different query arrays: each call's query order stays whole until
the call has walked by it, although the other thread's calls replace it in the tree's cache meanwhile."""
import threading

import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax
from paper_2507_23700_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_two_threads_replace_each_others_order():
    g = np.random.default_rng(21)
    data = inputs.cube(20_000, 3, g)
    r = float(inputs.radius_cube(len(data), 8.0))
    sets = [inputs.cube(9_000 + 500 * i, 3, g) for i in range(4)]
    tree = ax.arborx_bvh_build(torch.from_numpy(data).cuda())
    arrays = [torch.from_numpy(q).cuda() for q in sets]
    torch.cuda.synchronize()
    got = [[], []]

    def ask(who):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for turn in range(12):
                i = 2 * who + turn % 2
                off, idx = ax.arborx_query_spatial(tree, arrays[i], r)
                got[who].append((i, off, idx, *ax.arborx_query_knn(tree, arrays[i], 4)))
        stream.synchronize()

    threads = [threading.Thread(target=ask, args=(who,)) for who in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    want = [(*oracle.spatial(data, q, r), *oracle.knn(data, q, 4)) for q in sets]
    assert all(len(answers) == 12 for answers in got)
    for i, *answers in got[0] + got[1]:
        for a, w in zip(answers, want[i]):
            assert np.array_equal(a.cpu().numpy(), w), i
