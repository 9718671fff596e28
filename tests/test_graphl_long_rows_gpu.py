"""Descents of small graphs with rows of several items: the same bits in one
launch and in one per step, and no restart count much slower than another."""
import time

import numpy as np
import pytest
import torch

from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _star(n, extra=0):
    rng = np.random.default_rng(n)
    u = np.concatenate([np.zeros(n - 1, int), rng.integers(1, n, extra)])
    v = np.concatenate([np.arange(1, n), rng.integers(1, n, extra)])
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique(lo[lo != hi].astype(np.int64) * n + hi[lo != hi])
    return synth.csr_from_edges(n, key // n, key % n, np.where(rng.random(key.size) < 0.8, 1, -1))


@pytest.mark.parametrize("R", [1, 2, 3, 4, 8, 16, 32, 64])
@pytest.mark.parametrize("n,extra", [(1025, 0), (1026, 500), (2360, 0), (4000, 12000)])
def test_descent_equals_its_steps(n, extra, R):
    g = _star(n, extra)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=16)
    a = torch.rand(n, R, device="cuda", generator=torch.Generator("cuda").manual_seed(R)) * 2 - 1
    b = a.clone()
    for _ in range(7):
        b = G.graphl_step(b, 0.001)
    out = G.graphl_descend(a, 7)
    out = out[0] if isinstance(out, tuple) else out
    assert torch.equal(out, b)
    G.close()


def _us(g, R, steps=50):
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=16)
    a = torch.rand(len(g.row_ptr) - 1, R, device="cuda") * 2 - 1
    best = 1e9
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        G.graphl_descend(a, steps)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    G.close()
    return 1e6 * best


@pytest.mark.parametrize("n", [2360, 4000])
def test_few_restarts_are_not_slower_than_many(n):
    g = _star(n)
    assert max(_us(g, 1), _us(g, 4)) < 1.5 * _us(g, 32)
