"""Descents of small graphs with rows on both sides of what the registers hold:
the same bits as their steps, and the kernel that each takes."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _graph(n, longest, parts=3):
    """`parts` random trees of n / parts vertices, each with a vertex of degree `longest`."""
    rng = np.random.default_rng(n + longest)
    k = n // parts
    u, v = [], []
    for a in range(0, k * parts, k):
        u += [a + np.maximum(1, rng.random(k - 2) * np.arange(1, k - 1)).astype(int), np.full(longest, a)]
        v += [a + np.arange(2, k), a + 1 + np.arange(longest)]
    u, v = np.concatenate(u), np.concatenate(v)
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique(lo[lo != hi].astype(np.int64) * n + hi[lo != hi])
    return synth.csr_from_edges(n, key // n, key % n, np.where(rng.random(key.size) < 0.8, 1, -1))


@pytest.mark.parametrize("n,longest", [(900, 32), (900, 33), (900, 256), (900, 257), (1500, 24), (1500, 25), (1500, 100),
                                       (3000, 16), (3000, 17), (3000, 40)])
def test_descent_equals_its_steps(n, longest):
    g = _graph(n, longest)
    assert np.diff(g.row_ptr).max() == longest
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=16)
    for R in (1, 3, 32):
        a = torch.rand(n, R, device="cuda", generator=torch.Generator("cuda").manual_seed(R)) * 2 - 1
        b = a.clone()
        for _ in range(6):
            b = G.graphl_step(b, 0.001)
        assert torch.equal(G.graphl_descend(a, 6)[0], b)
    G.close()


def _kernels(n, longest):
    g = _graph(n, longest)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=16)
    a, out = torch.rand(n, 32, device="cuda") * 2 - 1, torch.empty(n, 32, device="cuda")
    G.graphl_descend(a, 6, out=out)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        G.graphl_descend(a, 6, out=out)
    hip, count = ctypes.CDLL("libamdhip64.so"), ctypes.c_size_t(64)
    nodes, params = (ctypes.c_void_p * 64)(), (ctypes.c_uint64 * 32)()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), nodes, ctypes.byref(count)) == 0
    found = set()
    for node in nodes[: count.value]:
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), params) == 0
        found.add(params[3])  # the function: behind the block (12 bytes, and 4) and a pointer
    G.close()
    return found


@pytest.mark.parametrize("n,held", [(900, 32), (1500, 24), (3000, 16)])
def test_kernel_by_the_longest_row(n, held):
    # rows past the registers take the kernel of graphs with long rows: without their
    # code the compiler keeps fewer reads in flight (500 steps of 1,413 vertices with
    # rows of 148: 2,295 us in the other one, 1,803 in this)
    assert _kernels(n, held + 1) == _kernels(n, 257) != _kernels(n, held)
