"""Forests under the default node format: trees whose frames differ (one step, float nodes, one point,
none), queries inside and outside of them, batches that packets of queries and workgroups straddle."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def trees(dim, rng):
    unit = rng.random((400, dim), dtype=np.float32)
    stretch = np.ones(dim, np.float32)
    stretch[0] = 1e5  # no common step: float nodes
    return [unit, unit[:0], unit[:1], unit * stretch, unit[:2], np.full((70, dim), 0.5, np.float32),
            (unit - np.float32(0.5)) * np.float32(3), unit[:65] * np.float32(0.1) + np.float32(2)]


@pytest.mark.parametrize("dim", [2, 3, 6])
@pytest.mark.parametrize("sizes", ["ones", "ragged", "wide", "many"])
def test_forest_of_mixed_frames(dim, sizes):
    rng = np.random.default_rng([dim, len(sizes)])
    vals = trees(dim, rng)
    toff = np.concatenate([[0], np.cumsum([len(v) for v in vals])]).astype(np.int64)
    values = np.ascontiguousarray(np.concatenate(vals), dtype=np.float32)
    T = len(vals)
    if sizes == "ones":
        per = np.ones(700, np.int64)
    elif sizes == "ragged":
        per = rng.integers(0, 40, 60)
    elif sizes == "wide":
        per = np.array([0, 257, 1, 600, 0, 0, 255])
    else:  # more batches than a 32-bit key holds beside the curve
        per = np.zeros((1 << 20) + 3, np.int64)
        per[rng.integers(0, len(per), 200)] = 3
        per[-1] = 2
    boff = np.concatenate([[0], np.cumsum(per)]).astype(np.int64)
    btree = rng.integers(0, T, len(per)).astype(np.int32)
    brad = rng.choice([0.05, 0.3, 2.0], len(per)).astype(np.float32)
    m = int(boff[-1])
    q = (rng.random((m, dim), dtype=np.float32) * np.float32(3) - np.float32(1)).astype(np.float32)
    used = [int(b) for b in np.flatnonzero(per)]
    fo = ax.arborx_forest_build(dev(values), toff)
    dq, bo, bt, br = dev(q), dev(boff), dev(btree), dev(brad)
    oc, os_ = np.zeros(m, np.int32), np.zeros(m, np.int64)
    for b in used:
        sl = slice(boff[b], boff[b + 1])
        oc[sl], os_[sl] = oracle.reduce(vals[btree[b]], q[sl], brad[b], dim=dim)
    for nq in (0, 1, 2):
        ax.arborx_set_tuning_op(ax.OP_REDUCE, queries_per_thread=nq, node_format=1) if nq else None
        try:
            c, s = ax.arborx_forest_query_reduce(fo, dq, bo, bt, br, ax.COUNT_SUMDIST)
        finally:
            ax.arborx_reset_tuning()
        assert np.array_equal(c.cpu().numpy(), oc) and np.array_equal(s.cpu().numpy(), os_), nq
    for k in (1, 8):
        od2, oix = np.zeros((m, k), np.float32), np.zeros((m, k), np.int32)
        for b in used:
            sl = slice(boff[b], boff[b + 1])
            od2[sl], oix[sl] = oracle.knn(vals[btree[b]], q[sl], k, dim=dim)
        d2, ix = ax.arborx_forest_query_knn(fo, dq, bo, bt, k)
        assert np.array_equal(ix.cpu().numpy(), oix) and np.array_equal(d2.cpu().numpy(), od2), k
