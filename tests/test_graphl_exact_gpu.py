"""graphL's row classes on whole numbers, where every float32 sum is exact in any
order: an entry lost, doubled or given to a wrong row shows as a difference.
Graphs whose rows end and begin where the classes do, for every lane layout."""
import numpy as np
import pytest
import torch

from oracle import graphl as ogl
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _hubs(pool, chords, degrees):
    """Rows of the given degrees over `pool` vertices that a cycle and random
    chords join, and three vertices without edges."""
    rng = np.random.default_rng(pool)
    a = np.arange(pool)
    x = rng.integers(0, pool, chords)
    us = [a, x] + [np.full(d, pool + i) for i, d in enumerate(degrees)]
    vs = [(a + 1) % pool, (x + 2 + rng.integers(0, pool - 4, chords)) % pool]
    vs += [rng.choice(pool, d, replace=False) for d in degrees]
    u, v = np.concatenate(us), np.concatenate(vs)
    u, v = np.minimum(u, v), np.maximum(u, v)
    key = np.unique((u.astype(np.int64) << 32 | v)[u != v])
    u, v = key >> 32, key & 0xFFFFFFFF
    return synth.csr_from_edges(pool + len(degrees) + 3, u, v, np.where(rng.random(u.size) < 0.6, 1, -1))


def _around(mid):
    return (1, 7, 8, 9, mid - 1, mid, mid + 1, 255, 256, 257, 1023, 1024, 1025, 2048, 2049, 2500)


# rows of more than `mid` entries take a wave each: 48 up to 8,192 vertices, else
# three times the mean length, at least 64 and at most 256
GRAPHS = {
    "few_vertices": (48, lambda: _hubs(3000, 3000, _around(48))),
    "mean_below": (64, lambda: _hubs(9000, 30000, _around(64))),
    "mean": (87, lambda: _hubs(9000, 114800, _around(87))),
    "mean_above": (256, lambda: _hubs(8300, 370000, _around(256))),
}


@pytest.fixture(scope="module", params=list(GRAPHS))
def graph(request):
    mid, make = GRAPHS[request.param]
    g = make()
    mean = int(g.row_ptr[-1]) // g.n
    assert mid == (48 if g.n <= 8192 else max(64, min(3 * mean, 256)))
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    yield g, G
    G.close()


@pytest.mark.parametrize("R", [1, 3, 4, 7, 8, 16, 20, 32, 33, 64])
def test_rows_are_exact_on_whole_numbers(graph, R):
    g, G = graph
    # odd, so that no entry is zero; sums of 2,500 of them, and squares of
    # them, stay far below 2^24
    x = 2.0 * np.random.default_rng(R).integers(-4, 4, (g.n, R)) + 1.0
    gamma = torch.from_numpy(x.astype(np.float32)).cuda()
    want = ogl.grad(g, x)
    assert np.array_equal(G.graphl_backward(gamma).cpu().numpy(), want)
    assert np.array_equal(G.graphl_forward(gamma).cpu().numpy(), ogl.loss(g, x))
    assert np.array_equal(G.graphl_step(gamma, 2.0).cpu().numpy(), x - 2.0 * want)
    # the descent's pass keeps scales: two steps of whole numbers below 2^24
    two, scales = G.graphl_descend(gamma, 2, 2.0)
    x1 = x - 2.0 * want
    x2 = x1 - 2.0 * ogl.grad(g, x1)
    assert np.abs(x2).max() < 2**24 and not scales().any()
    assert np.array_equal(two.cpu().numpy(), x2)
