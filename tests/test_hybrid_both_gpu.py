"""Hybrid sweeps: both kinds of trees in one launch and in two, in LDS and in
workspace slots, against the oracle; neither kind waits for the other."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _graph(n, parts, degree):
    """`parts` random trees with more edges among each one's vertices."""
    rng = np.random.default_rng(n + parts)
    cut = np.linspace(0, n, parts + 1).astype(int)
    u, v = [], []
    for a, b in zip(cut[:-1], cut[1:]):
        k = b - a
        u += [a + (rng.random(k - 1) * np.arange(1, k)).astype(int), rng.integers(a, b, k * degree)]
        v += [a + np.arange(1, k), rng.integers(a, b, k * degree)]
    u, v = np.concatenate(u), np.concatenate(v)
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique(lo[lo != hi].astype(np.int64) * n + hi[lo != hi])
    return synth.csr_from_edges(n, key // n, key % n, np.where(rng.random(key.size) < 0.7, 1, -1))


# the CSR in LDS, with one component and with several; links; slots with the stack
# in LDS and in memory; the most trees of one launch and more
@pytest.mark.parametrize("n,parts,degree,trees", [
    (1, 1, 0, 5), (30, 1, 2, 1), (30, 1, 2, 1200), (30, 1, 2, 3000), (30, 6, 1, 1000), (30, 6, 1, 2500), (300, 1, 3, 70),
    (300, 20, 2, 600), (4000, 1, 8, 5), (9000, 3, 2, 4), (11500, 1, 0, 6), (11500, 40, 2, 6), (70000, 1, 1, 3),
    (70000, 9, 1, 3)])
def test_hybrid_against_the_oracle(n, parts, degree, trees):
    g = _graph(n, parts, degree)
    ref = oracle.sweep(g, 9, 0, trees, checks=False, sampler="hybrid")
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * trees)
    G.set_sampler("hybrid")
    for schedule in (dict(), dict(path=2), dict(path=2, block=512), dict(grid=3)):
        G.set_schedule(**schedule)
        G.cloud_reset()
        sw = G.sweep_range(0, trees, 9, tree_switches=True).cpu().numpy().astype(np.uint64)
        assert np.array_equal(sw, ref.trees[:, 0]) and np.array_equal(G.cloud(), ref.cloud), schedule
    G.set_schedule()
    for t in range(min(trees, 3)):
        words, switches = G.tree_state(9, t)
        assert switches == ref.trees[t, 0]
        assert G.count(torch.from_numpy(words.view(np.int64)).cuda())[0].item() == switches
    G.close()


def test_hybrid_replays():
    g = _graph(300, 1, 3)
    ref = oracle.sweep(g, 9, 0, 200, checks=False, sampler="hybrid")
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=512)
    G.set_sampler("hybrid")
    G.sweep(200, 9)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        G.sweep(200, 9, stream=side)
    for _ in range(3):
        G.cloud_reset()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(G.cloud(), ref.cloud)
    G.close()


def test_neither_kind_waits_for_the_other():
    a = np.arange(2000)
    g = synth.csr_from_edges(2000, a[:-1], a[1:], np.ones(1999, int))
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=256)

    def us(sampler):
        G.set_sampler(sampler)
        best = 1e9
        for _ in range(12):
            G.cloud_reset()
            torch.cuda.synchronize()
            t = time.perf_counter()
            G.sweep(100, 3)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return 1e6 * best

    assert us("hybrid") < 1.35 * max(us("bfs"), us("rdfs"))
    G.close()
