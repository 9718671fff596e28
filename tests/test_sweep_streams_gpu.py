"""Sweeps of one handle under capture and on two streams at once, at the sizes
where the default schedule changes: whole numbers, so equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")

K = 800  # above three trees per CU


def _switches(g, seed):
    return oracle.sweep(g, seed, 0, K, checks=False).trees[:, 0]


# trees in LDS, of few edges and of many; trees in workspace memory
@pytest.mark.parametrize("n,m", [(6000, 30000), (5000, 110000), (20000, 60000)])
def test_captured_sweep_replays_match_oracle(n, m):
    g = synth.erdos_renyi_connected(n, m, 0.8, 3)
    ref = _switches(g, 11)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * K)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        out = G.sweep_range(0, K, 11, tree_switches=True, stream=side)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        out = G.sweep_range(0, K, 11, tree_switches=True, stream=side)
    for i in range(3):
        out.zero_()
        G.sweep(K, 12 + i)  # eager work between the replays
        G.cloud_reset()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().astype(np.uint64), ref), i
    G.status()
    G.close()


@pytest.mark.parametrize("n,m", [(6000, 30000), (5000, 110000)])
def test_sweeps_of_one_handle_on_two_streams(n, m):
    g = synth.erdos_renyi_connected(n, m, 0.8, 4)
    refs = [_switches(g, s) for s in (21, 22)]
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4 * K)
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    outs = []
    for _ in range(3):
        for s, seed in zip(streams, (21, 22)):
            with torch.cuda.stream(s):
                outs.append(G.sweep_range(0, K, seed, tree_switches=True, stream=s))
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        assert np.array_equal(out.cpu().numpy().astype(np.uint64), refs[i & 1]), i
    G.close()
