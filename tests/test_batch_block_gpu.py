"""The threads per workgroup of a batched sweep, read from a captured graph's
kernel nodes: the caller's, or the automatic schedule's for the default 256."""
import ctypes

import pytest
import torch

import oracle
from paper_2311_00869_amd import synth, tune

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")

hip = ctypes.CDLL("libamdhip64.so")


class _KernelNode(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint32 * 3), ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def _blocks(B, trees):
    """Threads per workgroup of the sweep's own kernels, between its reset and
    its summary (256 each)."""
    mn = torch.empty((B.G, 2), dtype=torch.int64, device="cuda")
    B.sweep_into(trees, 3, mn)
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=side):
        B.sweep_into(trees, 3, mn, stream=side)
    raw, count = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(count)) == 0
    out = []
    for node in nodes:
        p = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        out.append(p.block[0])
    assert len(out) == 3
    return sorted(out)


# a batch whose trees the automatic schedule sweeps alone in 256 threads, and
# one that it sweeps 64 at a time in 1,024
@pytest.mark.parametrize("graphs,n_lo,n_hi,trees,auto", [(300, 100, 300, 16, 256), (400, 2000, 9000, 64, 1024)])
def test_block_of_the_automatic_path(graphs, n_lo, n_hi, trees, auto):
    B = fr.BatchGraph(synth.config_batch(graphs, seed=6, n_lo=n_lo, n_hi=n_hi), cloud_capacity_per_graph=trees)
    assert _blocks(B, trees) == sorted([256, 256, auto])
    for block in (512, 1024):
        B.set_schedule(block=block)
        assert _blocks(B, trees) == [256, 256, block]
    for default in (dict(), dict(block=256), tune.default_batch_schedule(B)):
        B.set_schedule(**default)
        assert _blocks(B, trees) == sorted([256, 256, auto]), default
    B.close()


# batches of small graphs: trees alone; 64 at a time in narrow workgroups, for
# small graphs and for more of them than wide workgroups hold, and in wide ones
@pytest.mark.parametrize("graphs,n_lo,n_hi,trees,block", [
    (2000, 20, 200, 16, 256), (2000, 20, 200, 64, 256), (2000, 20, 200, 128, 256),
    (1000, 100, 400, 64, 1024), (1000, 100, 400, 128, 256)])
def test_automatic_block_of_small_graphs(graphs, n_lo, n_hi, trees, block):
    gs = synth.config_batch(graphs, seed=6, n_lo=n_lo, n_hi=n_hi)
    B = fr.BatchGraph(gs, cloud_capacity_per_graph=trees)
    assert _blocks(B, trees) == sorted([256, 256, block])
    mn, ds = (x.cpu().numpy() for x in B.sweep(trees, 3))
    for i in range(0, graphs, graphs // 5):
        r = oracle.sweep(gs[i], 3, 0, trees, checks=False)
        assert tuple(mn[i]) == r.best and ds[i] == len(r.cloud), i
    B.close()


def test_automatic_block_is_the_best_of_64_trees_at_a_time():
    B = fr.BatchGraph(synth.config_batch(2000, seed=6, n_lo=20, n_hi=200), cloud_capacity_per_graph=64)
    mn = torch.empty((B.G, 2), dtype=torch.int64, device="cuda")

    def ms(**schedule):
        B.set_schedule(**schedule)
        best = float("inf")
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            B.sweep_into(64, 5, mn)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert ms(path=0) <= 1.2 * min(ms(path=4, block=block) for block in (256, 512, 1024))
    B.close()
