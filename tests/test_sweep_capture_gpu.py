"""Statistics sweeps of a graph whose trees fit LDS under capture, between
eager sweeps of the same handle: whole numbers, so equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def test_captured_statistics_and_eager_sweeps():
    # trees in LDS: statistics take the multi-tree path, whose eager sweeps of
    # one handle take turns; a captured one stands in no line
    g = synth.erdos_renyi_connected(2000, 12000, 0.8, 5)
    trees, seed = 150, 9
    ref = oracle.sweep(g, seed, 0, trees, checks=False)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * trees)
    want = [x.clone() for x in G.sweep_stats(0, trees, seed)]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    minus = torch.zeros(g.n, dtype=torch.int64, device="cuda")
    switched = torch.zeros(g.m, dtype=torch.int64, device="cuda")

    def stats():
        G.sweep_stats(0, trees, seed, vertex_minus=minus, edge_switched=switched, stream=side)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        stats()
    for i in range(3):
        minus.zero_()
        switched.zero_()
        G.cloud_reset()
        G.sweep_stats(0, trees, seed + 1 + i)  # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(minus, want[0]) and torch.equal(switched, want[1]), i
    G.cloud_reset()
    got = G.sweep_stats(0, trees, seed)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert np.array_equal(G.cloud(), ref.cloud)
    G.close()


def test_sweeps_take_turns_across_a_capture():
    # eager statistics on one stream, a capture on another while they run, then
    # eager statistics on a third: the last ones wait for the first ones
    g = synth.erdos_renyi_connected(3000, 60000, 0.8, 6)
    trees = 1000
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=8 * trees)
    want = [[x.clone() for x in G.sweep_stats(0, trees, seed)] for seed in (1, 2)]
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    outs = [[torch.zeros_like(x) for x in want[0]] for _ in range(4)]
    torch.cuda.synchronize()
    for k in range(2):
        G.sweep_stats(0, trees, 1, *outs[2 * k], stream=streams[0])
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(streams[1]):
            graph.capture_begin(capture_error_mode="thread_local")
            G.sweep_stats(0, trees, 3, *[torch.zeros_like(x) for x in want[0]], stream=streams[1])
            graph.capture_end()
        G.sweep_stats(0, trees, 2, *outs[2 * k + 1], stream=streams[2])
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        for got, ref in zip(out, want[i & 1]):
            assert torch.equal(got, ref), i
    G.close()
