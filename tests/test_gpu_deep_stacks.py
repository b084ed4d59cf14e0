"""An explicit workgroup of 256 with 64 stack entries is launched with all of them: the rings and queues that the
walks over codes keep beside the stacks come on top.  The launches' LDS is read from a trace of the calls."""
import json

import numpy as np
import pytest

import oracle
import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WORD = 4 * 256  # bytes of one entry a thread


@pytest.mark.parametrize("dim", [2, 3, 6])
def test_every_entry_asked_for_is_there(dim, tmp_path):
    rng = np.random.default_rng(dim)
    pts = rng.random((3000, dim), dtype=np.float32)
    pts[:1500] *= np.float32(1e-3)  # long paths
    r = float(np.float32(0.6 * 3000 ** (-1.0 / dim)))
    d = torch.from_numpy(pts).cuda()
    ax.arborx_set_tuning(block=256, stack=64, node_format=1, queries_per_thread=1)
    try:
        t = ax.arborx_bvh_build(d)

        def calls():
            return (ax.arborx_query_spatial(t, d, r), ax.arborx_query_spatial_with_distances(t, d, r),
                    ax.arborx_dbscan(t, d, r, 4))

        calls()
        torch.cuda.synchronize()
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
            (off, idx), (off2, idx2, _), labels = calls()
            torch.cuda.synchronize()
    finally:
        ax.arborx_reset_tuning()
    out = str(tmp_path / "trace.json")
    p.export_chrome_trace(out)
    lds = {}
    for e in json.load(open(out))["traceEvents"]:
        kernel = e.get("args", {}).get("kernel", "")
        if "shared memory" in e.get("args", {}):
            for name in ("k_spatial_count", "k_pair_degree", "k_dbscan_pairs"):
                if name + "<" in kernel:
                    lds.setdefault(name, []).append(e["args"]["shared memory"])
    assert sorted(lds["k_spatial_count"]) == [(64 + 8) * WORD, (64 + 16) * WORD]  # without and with distances
    assert lds["k_pair_degree"] == [64 * WORD] and lds["k_dbscan_pairs"] == [(64 + 8) * WORD]
    o_off, o_idx = oracle.spatial(pts, pts, r, dim=dim)
    for a, b in ((off, idx), (off2, idx2)):
        assert np.array_equal(a.cpu().numpy(), o_off) and np.array_equal(b.cpu().numpy(), o_idx)
    assert np.array_equal(labels.cpu().numpy(), oracle.dbscan(pts, r, 4, dim=dim))
