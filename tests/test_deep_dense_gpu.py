"""Trees that reach most vertices in a few levels of many edges and the rest,
beside them or on a tail, in many levels of few: against the oracle, and in time."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _dense(n, degree, ring, near, tail):
    """`n` vertices of mean degree `degree`; a ring of `ring` with `near`
    neighbours on either side; a path of `tail` hung on the first part."""
    rng = np.random.default_rng(n)
    u, v = [rng.integers(0, n, n * degree // 2)], [rng.integers(0, n, n * degree // 2)]
    a = np.arange(ring)
    u += [n + a] * near
    v += [n + (a + j) % ring for j in range(1, near + 1)]
    b = n + ring + np.arange(tail)
    u.append(np.concatenate([[0], b[:-1]]) if tail else b)
    v.append(b)
    u, v, total = np.concatenate(u), np.concatenate(v), n + ring + tail
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique(lo[lo != hi].astype(np.int64) * total + hi[lo != hi])
    return synth.csr_from_edges(total, key // total, key % total, np.where(rng.random(key.size) < 0.8, 1, -1))


@pytest.mark.parametrize("shape,trees", [((5400, 40, 167, 5, 0), 1), ((5400, 40, 167, 5, 0), 6), ((5400, 40, 0, 0, 90), 6),
                                         ((1200, 40, 160, 2, 30), 300), ((9000, 12, 100, 2, 0), 3), ((900, 60, 0, 0, 0), 300)])
def test_dense_with_a_deep_part(shape, trees):
    g = _dense(*shape)
    few = min(trees, 6)
    ref = oracle.sweep(g, 7, 0, few, checks=False)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * trees)
    for block in (256, 512, 1024):
        G.set_schedule(path=1, block=block)
        sw = G.sweep_range(0, trees, 7, tree_switches=True).cpu().numpy().astype(np.uint64)
        assert np.array_equal(sw[:few], ref.trees[:, 0])
    G.set_schedule()
    G.cloud_reset()
    G.sweep_range(0, few, 7)
    assert np.array_equal(G.cloud(), ref.cloud)
    words, _ = G.tree_state(7, few - 1)
    assert G.count(torch.from_numpy(words.view(np.int64)).cuda())[0].item() == ref.trees[few - 1, 0]
    G.close()


def _us(g, trees):
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * trees)
    best = 1e9
    for _ in range(12):
        G.cloud_reset()
        torch.cuda.synchronize()
        t = time.perf_counter()
        G.sweep(trees, 3)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    G.close()
    return 1e6 * best


def test_a_deep_part_costs_its_own_levels():
    # the ring's 17 levels and more look at 800 edges, the dense part's at 108,000
    assert _us(_dense(5400, 40, 167, 5, 0), 64) < 1.8 * _us(_dense(5400, 40, 0, 0, 0), 64)
