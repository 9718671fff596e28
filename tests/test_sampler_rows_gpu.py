"""Randomized DFS over rows longer than a wave, at the lengths where the scan
changes, against the oracle; a hub's scan takes as long as its row."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _hub(d, extra):
    """A hub of degree `d` whose leaves have `extra` edges among themselves."""
    rng = np.random.default_rng(d)
    u = np.concatenate([np.zeros(d, int), rng.integers(1, d + 1, extra)])
    v = np.concatenate([np.arange(1, d + 1), rng.integers(1, d + 1, extra)])
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique(lo[lo != hi].astype(np.int64) * (d + 1) + hi[lo != hi])
    return synth.csr_from_edges(d + 1, key // (d + 1), key % (d + 1), np.where(rng.random(key.size) < 0.7, 1, -1))


@pytest.mark.parametrize("extra", [0, 40])
@pytest.mark.parametrize("d", [63, 64, 65, 128, 129, 192, 193, 255, 256, 257, 512, 513])
def test_rows_at_the_lengths_of_the_scan(d, extra):
    g = _hub(d, extra)
    ref = oracle.sweep(g, 3, 0, 70, checks=False, sampler="rdfs")
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=256)
    G.set_sampler("rdfs")
    for path in (1, 2):
        G.set_schedule(path=path)
        G.cloud_reset()
        sw = G.sweep_range(0, 70, 3, tree_switches=True).cpu().numpy().astype(np.uint64)
        assert np.array_equal(sw, ref.trees[:, 0]) and np.array_equal(G.cloud(), ref.cloud)
    G.close()


def _us(d):
    g = _hub(d, 0)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=256)
    G.set_sampler("rdfs")
    best = 1e9
    for _ in range(40):
        torch.cuda.synchronize()
        t = time.perf_counter()
        G.sweep(64, 3)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    G.close()
    return 1e6 * best


def test_a_hub_costs_its_row():
    # a leaf costs a scan of the hub, of one load and of two (2.75 times the time
    # for 1.7 times the leaves where every scan had eight)
    base = _us(1)
    assert _us(99) - base < 2.45 * (_us(59) - base)
