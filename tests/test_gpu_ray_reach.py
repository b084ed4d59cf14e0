"""Rays whose directions, origins or boxes sit where the multiplied slab test could round a hit away:
axis-parallel, tiny and huge components, origins on faces, far origins, boxes without extent."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def boxes(n, dim, rng, scale, shift):
    lo = np.floor(rng.random((n, dim)) * 16) / 16  # many equal planes
    ext = rng.choice([0.0, 1 / 16, 1 / 8, 0.3], size=(n, dim))
    b = np.stack([lo, lo + ext], axis=1) * scale + shift
    return np.ascontiguousarray(b, dtype=np.float32)


def rays(m, dim, b, rng, power):
    d = rng.standard_normal((m, dim)) * 10.0 ** rng.uniform(-power, power, size=(m, dim))
    d[rng.random((m, dim)) < 0.25] = 0.0  # axis-parallel, and some without a direction
    pick = b[rng.integers(0, len(b), m)]
    o = np.where(rng.random((m, dim)) < 0.5, pick[:, 0], pick[:, 1]).astype(np.float64)  # on planes of a box
    far = rng.random(m) < 0.3
    with np.errstate(over="ignore"):
        back = np.clip(d, -1e3, 1e3) * rng.uniform(0.5, 3.0, size=(m, 1))
        o[far] = (o - back)[far]  # aimed at a corner from outside
        return np.ascontiguousarray(np.stack([o, d], axis=1).astype(np.float32))


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("power", [0.0, 3.0, 29.0, 30.5, 37.9, 44.0])
@pytest.mark.parametrize("scale,shift", [(1.0, 0.0), (1e-20, 0.0), (3e15, -1e15), (1.0, 4096.0)])
def test_rays_at_the_edges_of_rounding(dim, power, scale, shift):
    rng = np.random.default_rng([dim, int(power * 10), int(abs(shift)) % 1000])
    b = boxes(600, dim, rng, scale, shift)
    r = rays(700, dim, b, rng, power)
    t = ax.arborx_bvh_build(dev(b), ax.BOXES)
    off, idx = ax.arborx_query_ray_intersect(t, dev(r))
    o_off, o_idx = oracle.ray_intersect(b, r, dim=dim, kind=oracle.BOXES)
    assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx)
    assert np.array_equal(ax.arborx_query_ray_count(t, dev(r)).cpu().numpy(), np.diff(o_off))
    for k in (1, 6):
        te, ix = ax.arborx_query_ray_nearest(t, dev(r), k)
        o_t, o_ix = oracle.ray_nearest(b, r, k, dim=dim, kind=oracle.BOXES)
        assert np.array_equal(ix.cpu().numpy(), o_ix) and np.array_equal(te.cpu().numpy(), o_t, equal_nan=True)
