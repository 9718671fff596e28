"""Several passes of the multi-tree sweep in flight at once, the rows a block
shares among its waves, and the small-row batches of short lists, against the
oracle."""
import numpy as np
import pytest

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu


def _graph(g, cap):
    from paper_2311_00869_amd import frustration as fr
    return fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=cap)


def _shared_rows():
    """Hubs whose rows sit on the boundaries of the shared rows and their
    parts (255, 256, 257, 383, 384, 385, 2047, 2048, 2049 edges) over one pool
    of 2,500 vertices, so that their neighbours overlap and many trees hit the
    same rows; the pool carries a cycle."""
    rng = np.random.default_rng(12)
    pool, us, vs = 2500, [], []
    for i, d in enumerate((255, 256, 257, 383, 384, 385, 2047, 2048, 2049)):
        leaves = rng.choice(pool, d, replace=False)
        us.append(np.full(d, pool + i))
        vs.append(leaves)
    a = np.arange(pool)
    us.append(a)
    vs.append((a + 1) % pool)
    u, v = np.concatenate(us), np.concatenate(vs)
    sign = np.where(rng.random(u.size) < 0.7, 1, -1)
    return synth.csr_from_edges(pool + 9, u, v, sign)


GRAPHS = {
    "shared_rows": _shared_rows,
    "medium": lambda: synth.chung_lu(30000, 100000, 2.3, 4, p_pos=0.85),
    # every component small or isolated: no big component to order by
    "pieces": lambda: synth.chung_lu(30000, 12000, 3.5, 5, p_pos=0.6),
}


# passes of 64 or 128 trees: one, two and four sets, ragged ones, more passes
# than sets (1,030 trees: 17 passes of 64, 9 of 128)
@pytest.mark.parametrize("name,trees", [("shared_rows", 65), ("shared_rows", 1030), ("medium", 129),
                                        ("medium", 300), ("pieces", 260)])
def test_passes_in_flight_match_oracle(name, trees):
    g = GRAPHS[name]()
    seed = 41
    ref = oracle.sweep(g, seed, 0, trees, checks=False)
    G = _graph(g, cap=trees)
    for s in [dict(path=0), dict(path=4, block=1024), dict(path=5, block=512), dict(path=5, block=1024),
              dict(path=5, block=1024, grid=3)]:
        G.set_schedule(**s)
        G.cloud_reset()
        sw = G.sweep_range(0, trees, seed, tree_switches=True).cpu().numpy().astype(np.uint64)
        assert np.array_equal(sw, ref.trees[:, 0]), s
        assert np.array_equal(G.cloud(), ref.cloud), s
        assert G.min_frustration() == ref.best, s
    G.close()


def test_statistics_of_passes_in_flight_add_up():
    # several sets add to the same counters; one pass at a time owns them
    g = GRAPHS["medium"]()
    trees, seed = 600, 9
    G = _graph(g, cap=trees)
    G.set_schedule(path=5, block=1024, grid=64)
    want = [x.cpu().numpy() for x in G.sweep_stats(0, trees, seed)]
    for s in (dict(path=0), dict(path=4, block=1024), dict(path=5, block=1024)):
        G.set_schedule(**s)
        G.cloud_reset()
        got = [x.cpu().numpy() for x in G.sweep_stats(0, trees, seed)]
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), s
    G.close()


@pytest.mark.parametrize("n,m,trees", [(1000, 5000, 256), (1000, 5000, 257), (1000, 5000, 800),
                                       (6000, 50000, 767), (6000, 50000, 768), (10300, 30000, 40)])
def test_automatic_schedule_by_tree_count(n, m, trees):
    # one tree per workgroup at its three widths, and on either side of the
    # tree count (three per CU of 256) that takes the multi-tree path
    g = synth.chung_lu(n, m, 2.3, 8, p_pos=0.8)
    seed = 3
    ref = oracle.sweep(g, seed, 0, trees, checks=False)
    G = _graph(g, cap=trees)
    sw = G.sweep_range(0, trees, seed, tree_switches=True).cpu().numpy().astype(np.uint64)
    assert np.array_equal(sw, ref.trees[:, 0])
    assert np.array_equal(G.cloud(), ref.cloud)
    G.close()


def test_automatic_schedule_on_a_deep_graph():
    # a 2 x 10,000 ladder is past the LDS limit, and its BFS trees are
    # thousands of levels deep: one tree per workgroup
    rng = np.random.default_rng(3)
    L = 10000
    a = np.arange(L)
    us = np.concatenate([a[:-1], a[:-1] + L, a])
    vs = np.concatenate([a[1:], a[1:] + L, a + L])
    g = synth.csr_from_edges(2 * L, us, vs, np.where(rng.random(us.size) < 0.8, 1, -1))
    trees, seed = 70, 6
    ref = oracle.sweep(g, seed, 0, trees, checks=False)
    G = _graph(g, cap=trees)
    sw = G.sweep_range(0, trees, seed, tree_switches=True).cpu().numpy().astype(np.uint64)
    assert np.array_equal(sw, ref.trees[:, 0])
    assert np.array_equal(G.cloud(), ref.cloud)
    G.close()


@pytest.mark.parametrize("graphs,n_hi,trees", [(3, 400, 15), (3, 4000, 33), (5, 4000, 100), (40, 4000, 65),
                                               (140, 4000, 17)])
def test_batch_automatic_schedule(graphs, n_hi, trees):
    # one tree per workgroup, trees of few graphs cut into groups (33 trees:
    # the last group shorter), whole groups of 64, and more graphs than half
    # the CUs
    from paper_2311_00869_amd import frustration as fr
    gs = synth.config_batch(graphs, seed=6, n_lo=20, n_hi=n_hi)
    seed = 77
    B = fr.BatchGraph(gs, cloud_capacity_per_graph=trees)
    mn, ds = B.sweep(trees, seed)
    mn, ds = mn.cpu().numpy(), ds.cpu().numpy()
    for i in range(0, graphs, max(1, graphs // 12)):
        r = oracle.sweep(gs[i], seed, 0, trees, checks=False)
        assert tuple(mn[i]) == r.best and ds[i] == len(r.cloud), i
        assert np.array_equal(B.cloud(i), r.cloud), i
    B.close()
