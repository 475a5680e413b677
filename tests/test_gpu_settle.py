"""The phases that turn picks into blocks, at the sizes where they can go wrong: hops of no picks, of exactly one tile of 1,024
slots and one slot more, of more tiles than a workgroup of the emit phase scans by itself (1,024), and of more tiles than
one look-back block (4,096); blocking steps (one launch per hop, workgroups hand offsets on) and steps in flight (mark and
emit phases); growing batches, whose grids are sized by an estimate that is too small at first."""
import numpy as np
import pytest

from oracle import gsso
from paper_2406_17918_amd import synth
from parity_util import run_parity, run_parity_pipelined, gpu_sampler, oracle_sampler, assert_blocks_equal

pytestmark = pytest.mark.gpu


def ring_graph(n, deg):
    """Node v's neighbors are v + 1 .. v + deg (mod n): every node has exactly `deg` of them."""
    indices = (np.arange(n, dtype=np.int64)[:, None] + np.arange(1, deg + 1)) % n
    indices.sort(axis=1)
    return synth.Graph([n], [synth.Relation(0, 0, np.arange(n + 1, dtype=np.int32) * deg, indices.astype(np.int32).reshape(-1))])


@pytest.mark.parametrize("batch,fan", [(0, [4]), (1, [1]), (255, [4, 4]), (256, [4, 4]), (257, [4, 4]), (1024, [1, 1]), (1025, [1, 1]),
                                       (16384, [64]), (16385, [64]), (65537, [64])])
@pytest.mark.parametrize("mode", [gsso.MODE_OTF, gsso.MODE_FBL])
def test_tile_edges(batch, fan, mode):
    g = ring_graph(max(200, batch + 77), 64 if fan[0] == 64 else 9)
    kw = dict(k=max(8, fan[0]), mode=mode, num_layers=len(fan), refresh_fraction=0.25, refresh_period=1, rng_seed=3)
    assert run_parity(g, kw, fan, batch, steps=range(2)) == run_parity_pipelined(g, kw, fan, batch, steps=range(2))


@pytest.mark.parametrize("blocking", [True, False])
def test_batches_that_outgrow_the_estimated_grid(blocking):
    # most seeds of the first steps have no neighbors: the estimate of later hops shrinks, then a batch fills its bound
    import torch
    n = 60000
    deg = np.zeros(n, np.int64); deg[: n // 2] = 9
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    indices = ((np.arange(n // 2)[:, None] * 7 + np.arange(1, 10) * 1001) % n).astype(np.int32)
    indices.sort(axis=1)
    g = synth.Graph([n], [synth.Relation(0, 0, indptr, indices.reshape(-1))])
    kw = dict(k=9, mode=gsso.MODE_FBL, num_layers=3, rng_seed=3)
    gs, os_ = gpu_sampler(g, kw), oracle_sampler(g, kw)
    for i in range(14):
        ids = np.arange(n // 2, n // 2 + 4000) if i < 12 else np.arange(4000)
        seeds = ids.astype(np.int32)
        dev = torch.from_numpy(seeds).cuda()
        if blocking:
            blocks = gs.step(dev, [5, 5, 9], i)
        else:
            gs.step_async(dev, [5, 5, 9], i)
            blocks = gs.step_wait()
        assert_blocks_equal(blocks, os_.step(seeds, [5, 5, 9], i), ctx=f"step {i}")
    gs.close(); os_.close()


@pytest.mark.parametrize("batch", [0, 3, 150, 900])
def test_typed_graph_blocking_and_pipelined(batch):
    g = synth.hetero_graph([1200, 2000, 60, 300], [(1, 2, 2600), (1, 0, 9000), (0, 0, 5000), (0, 3, 8000)], 2.2, seed=8)
    kw = dict(k=25, mode=gsso.MODE_OTF, num_layers=2, refresh_fraction=0.2, refresh_period=1, rng_seed=3)
    assert run_parity(g, kw, [25, 20], batch, steps=range(4)) == run_parity_pipelined(g, kw, [25, 20], batch, steps=range(4))
