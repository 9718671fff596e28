"""Launches of an exact count on both sides of the 320 workgroups (of 1,024
edges) up to which they add to the counts themselves, read from a captured
graph, and the counts of several groups of states against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


@pytest.mark.parametrize("m,launches", [(320 * 1024, 2), (320 * 1024 + 1, 3)])
def test_launches_of_a_group_of_states(m, launches):
    n, B = 3000, 130
    g = synth.erdos_renyi_connected(n, m, 0.7, 4)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    states = np.where(np.random.default_rng(3).random((B, n)) < 0.5, 1, -1).astype(np.int8)
    words = np.zeros((B, G.nwords), np.uint64)
    for b, s in enumerate(states):
        idx = np.flatnonzero(s < 0)
        np.bitwise_or.at(words[b], idx // 64, np.left_shift(np.uint64(1), (idx % 64).astype(np.uint64)))
    bits = torch.from_numpy(words.view(np.int64)).cuda()
    want = [oracle.count(g, s) for s in states]
    assert G.count(bits).cpu().numpy().tolist() == want
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=side):
        got = G.count(bits, stream=side)
    hip, nodes = ctypes.CDLL("libamdhip64.so"), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    assert nodes.value == 1 + 3 * launches  # the tensor of counts, three groups of up to 64 states
    graph.instantiate()
    for _ in range(3):
        got.fill_(7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert got.cpu().numpy().tolist() == want
    G.close()
