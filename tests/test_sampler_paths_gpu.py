"""The randomized DFS and Kruskal samplers at the sizes where their data moves
(CSR, stack, marks and forest in LDS or in memory, the two edge lists or all
the edges) and at row lengths where a scan changes: whole numbers, so equal to
the oracle."""
import numpy as np
import pytest

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _rows(extra):
    """Hubs of 15 .. 2,049 edges over a cycle of 3,000 vertices with `extra`
    random chords."""
    rng = np.random.default_rng(5)
    pool = 3000
    a = np.arange(pool)
    us, vs = [a], [(a + 1) % pool]
    for i, d in enumerate((15, 16, 17, 18, 63, 64, 65, 66, 511, 512, 513, 2046, 2047, 2048, 2049)):
        us.append(np.full(d, pool + i))
        vs.append(rng.choice(pool, d, replace=False))
    x = rng.integers(0, pool, extra)
    us.append(x)
    vs.append((x + 2 + rng.integers(0, pool // 2 - 4, extra)) % pool)
    u, v = np.concatenate(us), np.concatenate(vs)
    key = np.unique(np.minimum(u, v).astype(np.int64) << 32 | np.maximum(u, v))
    u, v = key >> 32, key & 0xFFFFFFFF
    return synth.csr_from_edges(pool + 15, u, v, np.where(rng.random(u.size) < 0.7, 1, -1))


def _check(g, sampler, K, scheds):
    ref = oracle.sweep(g, 19, 0, K, checks=False, sampler=sampler)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * K)
    G.set_sampler(sampler)
    for sched in scheds:
        if sched:
            G.set_schedule(**sched)
        G.cloud_reset()
        sw = G.sweep_range(0, K, 19, tree_switches=True).cpu().numpy().astype(np.uint64)
        assert np.array_equal(sw, ref.trees[:, 0]), sched
        assert np.array_equal(G.cloud(), ref.cloud), sched
    G.close()


AUTO = [None]
BOTH = [None, dict(path=1, block=256), dict(path=2, block=512)]

RDFS = {
    "rows_in_lds": (lambda: _rows(0), 9, BOTH),
    "rows_with_links": (lambda: _rows(15000), 9, BOTH),
    "several_waves": (lambda: synth.erdos_renyi_connected(300, 900, 0.8, 1), 1200, BOTH),
    "links_several_per_cu": (lambda: synth.erdos_renyi_connected(10000, 11000, 0.8, 2), 300, BOTH),
    "no_links": (lambda: synth.complete_graph(4300, -1), 1, AUTO),
    "stack_lds_last": (lambda: synth.erdos_renyi_connected(65536, 70000, 0.8, 3), 3, AUTO),
    "stack_memory": (lambda: synth.erdos_renyi_connected(65537, 70000, 0.8, 3), 3, AUTO),
    "marks_memory": (lambda: synth.erdos_renyi_connected(655424, 655600, 0.8, 4), 2, AUTO),
    "components": (lambda: synth.random_small(5000, 4000, 6, p_pos=0.6), 9, BOTH),
    "empty": (lambda: synth.isolated_vertices(0), 3, AUTO),
    "edgeless": (lambda: synth.isolated_vertices(130), 3, BOTH),
}


@pytest.mark.parametrize("name", RDFS)
def test_rdfs_paths(name):
    make, K, scheds = RDFS[name]
    _check(make(), "rdfs", K, scheds)


# n, m: the last n in LDS and the first beyond, the last with its forest in
# LDS and the first beyond, one list and two, and so many edges that the second
# list does not hold them
@pytest.mark.parametrize("n,m,K", [(8192, 20000, 9), (8193, 20000, 9), (8500, 10625, 9), (8500, 10626, 300),
                                   (36864, 80000, 5), (36865, 80000, 5), (2000, 60000, 300),
                                   (700, 120000, 9)])
def test_kruskal_paths(n, m, K):
    _check(synth.erdos_renyi_connected(n, m, 0.8, n), "kruskal", K, [None] + [dict(path=2, block=b) for b in (256, 512, 1024)])


@pytest.mark.parametrize("g", [synth.isolated_vertices(0), synth.isolated_vertices(130), _rows(0),
                               synth.random_small(5000, 9000, 6, p_pos=0.6)],
                         ids=["empty", "edgeless", "rows", "components"])
def test_kruskal_small_and_components(g):
    _check(g, "kruskal", 5, BOTH if g.n else AUTO)  # (an empty graph has no slots)
