"""The automatic block of BFS sweeps in LDS, read from a captured graph, on both
sides of the size where it turns, against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


@pytest.mark.parametrize("n,trees,block", [(2, 1, 256), (128, 64, 256), (128, 700, 256), (129, 64, 1024), (129, 700, 512)])
def test_block_of_small_sweeps(n, trees, block):
    g = synth.random_tree(2, 1) if n == 2 else synth.erdos_renyi_connected(n, 3 * n, 0.8, 4)
    ref = oracle.sweep(g, 5, 0, trees, checks=False)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * trees)
    sw = G.sweep_range(0, trees, 5, tree_switches=True).cpu().numpy().astype(np.uint64)
    assert np.array_equal(sw, ref.trees[:, 0]) and np.array_equal(G.cloud(), ref.cloud)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        G.sweep(trees, 5, stream=side)
    hip, count = ctypes.CDLL("libamdhip64.so"), ctypes.c_size_t(1)
    node, params = ctypes.c_void_p(), (ctypes.c_uint32 * 64)()  # blockDim comes first
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.byref(node), ctypes.byref(count)) == 0
    assert count.value == 1 and hip.hipGraphKernelNodeGetParams(node, params) == 0
    assert params[0] == block
    G.close()
