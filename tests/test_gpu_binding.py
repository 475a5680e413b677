"""The binding's native calls make the same tensors as its Python view of the raw blocks: a block's arrays share the
allocation the library wrote them to, empty ones included, and an allocator may make its own views."""
import numpy as np
import pytest

from oracle import gsso
from paper_2406_17918_amd import synth
from parity_util import oracle_sampler, assert_blocks_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("own_views", [False, True])
@pytest.mark.parametrize("batch", [0, 1, 100])
def test_native_blocks_equal_the_views_of_the_raw_blocks(own_views, batch):
    import torch
    from paper_2406_17918_amd import gss

    class OwnViews(gss._TorchAllocator):
        def view_i32(self, ptr, n):
            return super().view_i32(ptr, n)

    g = synth.hetero_graph([300, 500, 20, 60], [(1, 2, 600), (1, 0, 2000), (0, 0, 1000), (0, 3, 2000)], 2.2, seed=8)
    kw = dict(k=8, mode=gsso.MODE_OTF, num_layers=2, refresh_fraction=0.25, refresh_period=1, rng_seed=3)
    a = OwnViews("cuda:0") if own_views else gss._TorchAllocator("cuda:0")
    s, o = gss.Sampler(g.num_nodes, gss.upload_graph(g), allocator=a, **kw), oracle_sampler(g, kw)
    seeds = synth.seeds_for_step(300, batch, 4, 0)
    s.step_async(torch.from_numpy(seeds).cuda(), (4, 5), 0)
    raw = s.step_wait_raw()
    want = s._wrap(raw)
    assert_blocks_equal(want, o.step(seeds, [4, 5], 0))
    blocks = s.step(torch.from_numpy(seeds).cuda(), [4, 5], 1)
    assert_blocks_equal(blocks, o.step(seeds, [4, 5], 1))
    for b in blocks:
        for t in b.src_nodes + b.src_local + b.dst_local:
            assert t.dtype == torch.int32 and t.is_cuda and t.is_contiguous()
            assert t.numel() == 0 or t.untyped_storage().data_ptr() in a.live
    s.close(); o.close()
    if batch:                              # the tensors keep their memory after the sampler is gone
        assert int(blocks[1].src_nodes[0][0]) == int(seeds[0])
