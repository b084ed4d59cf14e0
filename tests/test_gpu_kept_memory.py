"""A program that needs the memory the library keeps free asks for it by naming the default allocator, also
while structures of its own live (the call is refused then, but the blocks go back)."""
import gc

import pytest

import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("live", [False, True])
def test_kept_blocks_go_back_on_request(live):
    d = torch.rand((3_000_000, 3), device="cuda")
    small = ax.arborx_bvh_build(d[:1000].contiguous()) if live else None
    t = ax.arborx_bvh_build(d)
    ax.arborx_query_knn(t, d[:1000].contiguous(), 4)
    del t
    gc.collect()
    torch.cuda.synchronize()
    kept = torch.cuda.mem_get_info()[0]
    if live:
        with pytest.raises(Exception):
            ax.arborx_set_allocator()
    else:
        ax.arborx_set_allocator()
    assert torch.cuda.mem_get_info()[0] >= kept + 3_000_000 * 64  # the nodes at least
    del small
