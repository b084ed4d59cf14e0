"""Sphere walks in the codes of a tree's frame: the cases where rounding of the frame, the query or
the radius could prune a match.  Every result is compared with the oracle element by element."""
import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def frames(dim, n, rng):
    """(name, points, scale of a typical neighbour distance)."""
    unit = rng.random((n, dim), dtype=np.float32)
    h = n ** (-1.0 / dim)
    for ratio in (100.0, 300.0, 1e5):  # one step up to 256, float nodes beyond
        stretch = np.ones(dim, np.float32)
        stretch[0] = ratio
        yield f"stretched {ratio:g}", unit * stretch, h * ratio ** (1.0 / dim)
    yield "far from the origin", unit + np.float32(3.0e5), max(h, 0.04)
    yield "straddling zero, large", (unit - np.float32(0.5)) * np.float32(1e18), h * 1e18
    yield "tiny", unit * np.float32(1e-36), h * 1e-36
    yield "denormal", unit * np.float32(1e-41), h * 1e-41
    flat = unit.copy()
    flat[:, -1] = 0.25  # no extent in one dimension
    yield "flat", flat, n ** (-1.0 / max(1, dim - 1))
    yield "one place", np.full((n, dim), 0.75, np.float32), 1.0
    lattice = np.floor(unit * 6).astype(np.float32)  # many equal points and equal distances
    yield "lattice", lattice, 1.0
    clump = unit.copy()
    clump[: n // 2] = np.float32(0.5) + (unit[: n // 2] - np.float32(0.5)) * np.float32(1e-4)  # inside one code
    yield "clump", clump, h


@pytest.mark.parametrize("dim", [2, 3, 6])
@pytest.mark.parametrize("n", [1, 2, 65, 1500])
def test_code_walks_match_the_oracle(dim, n):
    rng = np.random.default_rng([dim, n])
    for name, pts, scale in frames(dim, n, rng):
        pts = np.ascontiguousarray(pts, dtype=np.float32)
        lo, hi = pts.min(0), pts.max(0)
        q = [pts[rng.integers(0, n, 40)],                                                  # on the points
             (lo + (hi - lo) * rng.random((40, dim), dtype=np.float32)).astype(np.float32),
             np.nextafter(pts[rng.integers(0, n, 10)], np.float32(np.inf)),               # one ulp away
             np.stack([lo, hi]), np.stack([lo - np.float32(scale), hi + np.float32(scale)])]  # corners and outside
        q = np.ascontiguousarray(np.concatenate(q), dtype=np.float32)
        t = ax.arborx_bvh_build(dev(pts))
        dq = dev(q)
        for r in (0.0, 0.5 * scale, 1.5 * scale, np.inf):
            r = float(np.float32(r))
            o_off, o_idx = oracle.spatial(pts, q, r, dim=dim)
            off, idx = ax.arborx_query_spatial(t, dq, r)
            assert np.array_equal(off.cpu().numpy(), o_off) and np.array_equal(idx.cpu().numpy(), o_idx), (name, r)
            c, _ = ax.arborx_query_spatial_reduce(t, dq, r, ax.COUNT)
            assert np.array_equal(c.cpu().numpy(), np.diff(o_off)), (name, r)
            few = ax.arborx_query_spatial_count_up_to(t, dq, r, 2)
            assert np.array_equal(few.cpu().numpy(), np.minimum(np.diff(o_off), 2)), (name, r)
            if n <= 65 or r <= 0.5 * scale:
                deg = ax.arborx_self_join_degree(t, r).cpu().numpy()
                self_off, _ = oracle.spatial(pts, pts, r, dim=dim)
                assert np.array_equal(deg, np.diff(self_off) - 1), (name, r)
        for k in (1, 4, 10, 16, 40):
            o_d2, o_ix = oracle.knn(pts, q, k, dim=dim)
            d2, ix = ax.arborx_query_knn(t, dq, k)
            assert np.array_equal(ix.cpu().numpy(), o_ix) and np.array_equal(d2.cpu().numpy(), o_d2), (name, k)
