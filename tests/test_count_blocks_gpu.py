"""The exact count at the number of workgroups up to which they add to the
counts themselves, without a second launch, against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _words(states):
    out = np.zeros((states.shape[0], (states.shape[1] + 63) // 64), np.uint64)
    for b, s in enumerate(states):
        idx = np.flatnonzero(s < 0)
        np.bitwise_or.at(out[b], idx // 64, np.left_shift(np.uint64(1), (idx % 64).astype(np.uint64)))
    return out


# 1,024 edges to a workgroup: none, one, 64 and 65 of them
@pytest.mark.parametrize("n,m", [(70, 0), (300, 1023), (2000, 64 * 1024), (2000, 64 * 1024 + 1)])
@pytest.mark.parametrize("B", [1, 32, 33, 70])
def test_counts_around_the_second_launch(n, m, B):
    g = synth.erdos_renyi_connected(n, m, 0.7, 4) if m else synth.isolated_vertices(n)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    states = np.where(np.random.default_rng(B).random((B, n)) < 0.5, 1, -1).astype(np.int8)
    want = [oracle.count(g, s) for s in states]
    words = torch.from_numpy(_words(states).view(np.int64))
    R = min(B, 64)
    gamma = torch.from_numpy(np.ascontiguousarray(states[:R].T).astype(np.float32)).cuda()
    for _ in range(2):  # (the second time over counts that are there)
        assert G.count(words).cpu().numpy().tolist() == want
        assert G.round_count(gamma).cpu().numpy().tolist() == want[:R]
    G.close()


def test_a_small_graphs_rounded_count_takes_two_launches():
    g = synth.erdos_renyi_connected(1000, 5000, 0.8, 2)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    gamma = torch.from_numpy(synth.graphl_init(g.n, 64, 1)).cuda()
    want = G.round_count(gamma)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=side):
        got = G.round_count(gamma, stream=side)
    hip = ctypes.CDLL("libamdhip64.so")
    nodes = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    assert nodes.value == 2
    graph.instantiate()
    for _ in range(3):
        got.fill_(7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    G.close()
