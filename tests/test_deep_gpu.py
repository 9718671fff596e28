"""Deep graphs: trees of many levels, of which each holds little, in LDS and
beyond, alone and in a batch, against the oracle."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _csr(n, u, v):
    u, v = np.concatenate(u), np.concatenate(v)
    return synth.csr_from_edges(n, u, v, np.where(np.random.default_rng(n).random(u.size) < 0.7, 1, -1))


def _path(n):
    return _csr(n, [np.arange(n - 1)], [np.arange(1, n)])


def _ring(n, k):
    a = np.arange(n)
    return _csr(n, [a] * k, [(a + j) % n for j in range(1, k + 1)])


def _broom(handle, leaves, tail):
    """A path, a hub with `leaves` leaves at its end, and a path from every
    hundredth leaf."""
    u, v = [np.arange(handle - 1)], [np.arange(1, handle)]
    n = handle
    u.append(np.full(leaves, handle - 1))
    v.append(n + np.arange(leaves))
    ends, n = n + np.arange(0, leaves, 100), n + leaves
    for _ in range(tail):
        u.append(ends)
        v.append(n + np.arange(ends.size))
        ends, n = n + np.arange(ends.size), n + ends.size
    return _csr(n, u, v)


def _pieces():
    """A path, a ring, stars and vertices without edges."""
    u, v, n = [np.arange(299)], [np.arange(1, 300)], 300
    a = np.arange(100)
    u.append(n + a)
    v.append(n + (a + 1) % 100)
    n += 150
    for d in (1, 5, 200):
        u.append(np.full(d, n))
        v.append(n + 1 + np.arange(d))
        n += d + 3
    return _csr(n, u, v)


GRAPHS = {
    # roots at an end and inside, with as many vertices left after six levels
    # that these are just over and under the 16 levels like the last
    **{f"path_{n}": (lambda n=n: _path(n), 60) for n in (7, 8, 22, 23, 24, 25, 44, 45, 46, 60)},
    "ring": (lambda: _ring(2000, 5), 10),
    "ring_more_than_held": (lambda: _ring(9000, 10), 3),
    "broom": (lambda: _broom(30, 3000, 8), 12),
    "pieces": (_pieces, 20),
    "last_in_lds": (lambda: _path(10922), 2),
}


@pytest.mark.parametrize("name", GRAPHS)
def test_deep_trees_in_lds_match_oracle(name):
    make, K = GRAPHS[name]
    g = make()
    ref = oracle.sweep(g, 29, 0, K, checks=False)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * K)
    for block in (256, 512, 1024):
        G.set_schedule(path=1, block=block, grid=3)
        G.cloud_reset()
        sw = G.sweep_range(0, K, 29, tree_switches=True).cpu().numpy().astype(np.uint64)
        assert np.array_equal(sw, ref.trees[:, 0]), block
        assert np.array_equal(G.cloud(), ref.cloud), block
    words, s = G.tree_state(29, 1)
    assert np.array_equal(words, oracle.canonical_words(g, oracle.tree(g, 29, 1, "bfs")[2]))
    assert s == int(ref.trees[1, 0])
    G.close()


def test_deep_batch_matches_oracle():
    graphs = [make() for make, _ in GRAPHS.values()] + [_path(15000)]
    K = 3
    ref = [oracle.sweep(g, 29, 0, K, checks=False) for g in graphs]
    B = fr.BatchGraph(graphs, cloud_capacity_per_graph=K)
    for block in (256, 512, 1024):
        B.set_schedule(path=1, block=block)
        least, distinct = B.sweep(K, 29)
        for i, r in enumerate(ref):
            assert tuple(least[i].tolist()) == r.best, (block, i)
            assert np.array_equal(B.cloud(i), r.cloud), (block, i)
            assert int(distinct[i]) == len(r.cloud)
    B.close()


def _sweep_ms(G, K, **schedule):
    G.set_schedule(**schedule)
    best = float("inf")
    for _ in range(4):
        G.cloud_reset()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        G.sweep(K, 5)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_a_deep_tree_in_lds_is_no_slower_than_in_memory():
    # 450 levels of 20 vertices and 200 edges, of 90,000 edges in all
    g = _ring(9000, 10)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=256)
    lds, memory = (_sweep_ms(G, 100, path=p, block=1024) for p in (1, 2))
    assert lds <= memory
    G.close()


def test_automatic_block_of_a_batch_of_deep_graphs():
    # eight trees of 300 small rings: little to do in a level, so narrow
    # workgroups, four to a CU
    B = fr.BatchGraph([_ring(1000, 5)] * 300, cloud_capacity_per_graph=8)

    def ms(**schedule):
        B.set_schedule(**schedule)
        best = float("inf")
        mn = torch.empty((B.G, 2), dtype=torch.int64, device="cuda")
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            B.sweep_into(8, 5, mn)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert ms(path=0) <= 1.25 * ms(path=1, block=256)
    B.close()


def _ladder(L):
    a = np.arange(L)
    return _csr(2 * L, [a[:-1], a[:-1] + L, a], [a[1:], a[1:] + L, a + L])


def _paths(c, L):
    a = np.arange(c * L).reshape(c, L)
    return _csr(c * L, [a[:, :-1].ravel()], [a[:, 1:].ravel()])


def _star_and_paths():
    """A star, the main component, and long paths beside it."""
    u, v, n = [np.zeros(12999, np.int64)], [np.arange(1, 13000)], 13000
    for _ in range(3):
        u.append(n + np.arange(1999))
        v.append(n + 1 + np.arange(1999))
        n += 2000
    return _csr(n, u, v)


def _path_and_stars():
    """A path, the main component, and stars beside it, whose hubs are the
    vertices of highest degree."""
    u, v, n = [np.arange(11999)], [np.arange(1, 12000)], 12000
    for _ in range(10):
        u.append(np.full(99, n))
        v.append(n + 1 + np.arange(99))
        n += 100
    return _csr(n, u, v)


# past LDS: the trees as deep as the graph's diameter, in its main component or
# beside it, above and below 20,000 in n + m / 2, with and without a component
# of more than 1,024 vertices
PAST_LDS = {
    "ladder": lambda: _ladder(5500), "cycle": lambda: synth.cycle_graph(13000, (0,)),
    "paths": lambda: _paths(20, 1000), "star_and_paths": _star_and_paths,
    "path_and_stars": _path_and_stars, "ring": lambda: _ring(12000, 6),
}
SHALLOW = {
    "er": lambda: synth.erdos_renyi_connected(11000, 30000, 0.8, 3),
    "stars": lambda: _csr(20000, [np.repeat(np.arange(0, 20000, 500), 499)],
                          [np.setdiff1d(np.arange(20000), np.arange(0, 20000, 500))]),
}


def _multi_passes(G, K):
    """Records of the multi-tree kernel's phase log over a sweep (0: another ran)."""
    log = G.phase_log(2048)
    G.cloud_reset()
    sw = G.sweep_range(0, K, 29, tree_switches=True).cpu().numpy().astype(np.uint64)
    records = int(log[0])
    G.phase_log(0)
    return records, sw


@pytest.mark.parametrize("name", [*PAST_LDS, *SHALLOW])
def test_deep_graphs_past_lds_keep_off_the_grid_barriers(name):
    deep = name in PAST_LDS
    g = (PAST_LDS if deep else SHALLOW)[name]()
    K = 40
    ref = oracle.sweep(g, 29, 0, K, checks=False)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=K)
    records, sw = _multi_passes(G, K)
    assert (records == 0) == deep
    assert np.array_equal(sw, ref.trees[:, 0])
    assert np.array_equal(G.cloud(), ref.cloud)
    G.close()


def test_a_deep_graph_uploads_without_its_whole_bfs():
    # past 135,000 in n + m / 2, where levels are counted for the tree order only,
    # that is made from 65,536 vertices on
    def ms(g):
        arrays = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (g.row_ptr, g.col, g.sign)]
        best = float("inf")
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            G = fr.Graph(*arrays, cloud_capacity=16)
            torch.cuda.synchronize()
            best = min(best, 1e3 * (time.perf_counter() - t))
            G.close()
        return best

    assert ms(_ring(60000, 4)) <= ms(_ring(70000, 4)) / 4
