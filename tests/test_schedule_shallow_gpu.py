"""The automatic path of graphs past LDS with few edges: about as fast as the
better of one tree per workgroup and many trees per pass."""
import time

import numpy as np
import pytest
import torch

from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _parts(sizes, edges, alone, seed):
    """Random trees of `sizes` vertices, `edges` more edges among them, and
    `alone` vertices without edges."""
    rng = np.random.default_rng(seed)
    u, v, n = [], [], 0
    for k in sizes:
        u.append(n + (rng.random(k - 1) * np.arange(1, k)).astype(int))
        v.append(n + np.arange(1, k))
        u.append(n + rng.integers(0, k, edges * k // sum(sizes)))
        v.append(n + rng.integers(0, k, edges * k // sum(sizes)))
        n += k
    u, v, n = np.concatenate(u), np.concatenate(v), n + alone
    p = rng.permutation(n)
    u, v = p[u], p[v]
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique(lo[lo != hi].astype(np.int64) * n + hi[lo != hi])
    return synth.csr_from_edges(n, key // n, key % n, np.where(rng.random(key.size) < 0.8, 1, -1))


def _us(G, trees, path):
    G.set_schedule(path=path, block=256 if path == 2 else 1024)
    if path == 0:
        G.set_schedule()
    best = 1e9
    for _ in range(12):
        G.cloud_reset()
        torch.cuda.synchronize()
        t = time.perf_counter()
        G.sweep(trees, 3)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return 1e6 * best


@pytest.mark.parametrize("sizes,edges,alone,trees", [((600, 480), 1800, 12100, 64), ((600, 480), 1800, 12100, 130),
                                                     ((6700, 1000, 430), 0, 9500, 130), ((14000,), 60000, 0, 100),
                                                     ((600, 480), 1800, 12100, 1000), ((14000,), 0, 0, 7)])
def test_path_of_shallow_graphs(sizes, edges, alone, trees):
    g = _parts(sizes, edges, alone, 3)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * trees)
    best = min(_us(G, trees, p) for p in (2, 4, 5))
    assert _us(G, trees, 0) < 1.15 * best
    G.close()
