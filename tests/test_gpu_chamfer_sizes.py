"""Chamfer pairs of empty, tiny and uneven clouds, around the workgroup sizes of its kernels.
Tolerances: sums are float64, each result rounded to float32 once (2^-24), so 2^-23 of the value and the
float64 rounding of the terms before cancellation."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("na,nb", [([1], [1]), ([0, 3, 1], [2, 0, 1]), ([255, 1, 257], [2, 300, 64]),
                                   ([8193, 40], [17, 9300])])
def test_forward_and_backward(na, nb):
    rng = np.random.default_rng([len(na), sum(na), sum(nb)])
    ao, bo = (np.concatenate([[0], np.cumsum(x)]).astype(np.int64) for x in (na, nb))
    a = rng.random((int(ao[-1]), 3), dtype=np.float32)
    b = (rng.random((int(bo[-1]), 3), dtype=np.float32) * np.float32(1.5) - np.float32(0.3)).astype(np.float32)
    loss, nab, nba = ax.arborx_chamfer_forward(dev(a), ao, dev(b), bo)
    o_loss, o_ab, o_ba = oracle.chamfer_forward(a, ao, b, bo)
    assert np.array_equal(nab.cpu().numpy(), o_ab) and np.array_equal(nba.cpu().numpy(), o_ba)
    assert np.allclose(loss.cpu().numpy(), o_loss, rtol=2.0 ** -23, atol=0)
    g = rng.standard_normal(len(na)).astype(np.float32)
    ga, gb = ax.arborx_chamfer_backward(dev(a), ao, dev(b), bo, nab, nba, dev(g))
    oga, ogb = oracle.chamfer_backward(a, ao, b, bo, o_ab, o_ba, g.astype(np.float64))
    for got, want in ((ga, oga), (gb, ogb)):
        assert np.allclose(got.cpu().numpy(), want, rtol=2.0 ** -23, atol=1e-11 * max(na + nb))
