"""Sweeps of one handle with different samplers on two streams at once, where
one keeps its trees in LDS and the other in workspace slots: whole numbers, so
equal to each sampler's sweep alone, whose first trees equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


# sizes where the CSR does not fit LDS and Kruskal's trees do not, but the
# randomized DFS's do; two sweeps of the DFS write the same links
@pytest.mark.parametrize("samplers", [("rdfs", "kruskal"), ("hybrid", "kruskal"), ("rdfs", "rdfs")])
def test_samplers_overlap_on_two_streams(samplers):
    n, m, K = 9000, 30000, 300
    g = synth.erdos_renyi_connected(n, m, 0.8, 7)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=10 * K)
    ref = {}
    for s in set(samplers):
        G.set_sampler(s)
        ref[s] = G.sweep_range(0, K, 21, tree_switches=True).cpu().numpy().astype(np.uint64)
        assert np.array_equal(ref[s][:6], oracle.sweep(g, 21, 0, 6, checks=False, sampler=s).trees[:, 0])
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = []
    for _ in range(3):
        for stream, sampler in zip(streams, samplers):
            G.set_sampler(sampler)
            with torch.cuda.stream(stream):
                outs.append((sampler, G.sweep_range(0, K, 21, tree_switches=True, stream=stream)))
    torch.cuda.synchronize()
    for i, (sampler, out) in enumerate(outs):
        assert np.array_equal(out.cpu().numpy().astype(np.uint64), ref[sampler]), (i, sampler)
    G.close()
