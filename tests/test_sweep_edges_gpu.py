"""The LDS sweep over the edges at the edges of what a thread holds, of the
vertices that fit and of the components, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu


def _grid(w, h):
    i = np.arange(w * h)
    r, d = i[i % w < w - 1], i[i < w * (h - 1)]
    u, v = np.concatenate([r, d]), np.concatenate([r + 1, d + w])
    return synth.csr_from_edges(w * h, u, v, np.where(np.random.default_rng(w).random(u.size) < 0.7, 1, -1))


GRAPHS = {
    "edge": (lambda: synth.random_tree(2, 1), 40),
    "edgeless": (lambda: synth.isolated_vertices(70), 5),
    "held_256": (lambda: synth.erdos_renyi_connected(300, 32 * 256, 0.8, 1), 40),
    "held_256_over": (lambda: synth.erdos_renyi_connected(300, 32 * 256 + 1, 0.8, 1), 40),
    "held_512_over": (lambda: synth.erdos_renyi_connected(1000, 32 * 512 + 7, 0.8, 2), 20),
    "held_1024": (lambda: synth.erdos_renyi_connected(2000, 32 * 1024, 0.8, 3), 10),
    "held_1024_over": (lambda: synth.erdos_renyi_connected(2000, 32 * 1024 + 1, 0.8, 3), 10),
    "last_in_lds": (lambda: synth.erdos_renyi_connected(10922, 30000, 0.8, 4), 10),
    "grid": (lambda: _grid(60, 20), 20),
    "path": (lambda: synth.cycle_graph(5000, (0, 7)), 5),
    "components": (lambda: synth.random_small(3000, 2600, 6, p_pos=0.6), 20),
    "pairs": (lambda: synth.csr_from_edges(200, np.arange(0, 200, 2), np.arange(1, 200, 2),
                                           np.where(np.arange(100) % 3 == 0, -1, 1)), 20),
    "hubs": (lambda: synth.chung_lu(4000, 20000, 2.1, 5, p_pos=0.7), 20),
}


@pytest.mark.parametrize("name", GRAPHS)
def test_edges_sweep_matches_oracle(name):
    from paper_2311_00869_amd import frustration as fr
    make, K = GRAPHS[name]
    g = make()
    ref = oracle.sweep(g, 23, 0, K, checks=False)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * K)
    for block in (256, 512, 1024):
        G.set_schedule(path=1, block=block, grid=3)  # several trees per workgroup
        G.cloud_reset()
        sw = G.sweep_range(0, K, 23, tree_switches=True).cpu().numpy().astype(np.uint64)
        assert np.array_equal(sw, ref.trees[:, 0]), block
        assert np.array_equal(G.cloud(), ref.cloud), block
    words, s = G.tree_state(23, 2)
    assert np.array_equal(words, oracle.canonical_words(g, oracle.tree(g, 23, 2, "bfs")[2]))
    assert s == int(ref.trees[2, 0])
    G.close()
