"""The randomized DFS of a graph of several components, which the waves of a
tree share: one to four of them, with the CSR in LDS and with links, beside the
hybrid's BFS trees; whole numbers, so equal to the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _pieces(sizes, chords):
    """A cycle with `chords` random chords for every size (a path below four),
    and a vertex without edges after each."""
    rng = np.random.default_rng(len(sizes))
    us, vs, n = [], [], 0
    for s in sizes:
        a = np.arange(s)
        u, v = (a, (a + 1) % s) if s > 3 else (a[:-1], a[1:])
        if s > 6:
            x = rng.integers(0, s, chords)
            u, v = np.concatenate([u, x]), np.concatenate([v, (x + 2 + rng.integers(0, s - 4, chords)) % s])
        key = np.unique(np.minimum(u, v).astype(np.int64) << 32 | np.maximum(u, v))
        us.append(n + (key >> 32))
        vs.append(n + (key & 0xFFFFFFFF))
        n += s + 1
    u, v = np.concatenate(us), np.concatenate(vs)
    return synth.csr_from_edges(n, u, v, np.where(rng.random(u.size) < 0.7, 1, -1))


GRAPHS = {
    "two": (lambda: _pieces([40, 40], 30), 6),
    "pairs": (lambda: _pieces([2] * 150, 0), 12),
    "giant_and_small": (lambda: _pieces([600] + [3, 5, 9] * 20, 400), 12),
    "links": (lambda: _pieces([3000, 2900, 2000, 50, 7], 9000), 4),
    "stack_in_slots": (lambda: _pieces([40000, 39000], 100), 2),
}


# trees per CU of 256: up to four, up to eight and more
@pytest.mark.parametrize("name,K", [(n, k) for n, (_, k) in GRAPHS.items()] + [("two", k) for k in (300, 1100, 2100)])
@pytest.mark.parametrize("sampler", ["rdfs", "hybrid"])
def test_components_match_oracle(name, K, sampler):
    g = GRAPHS[name][0]()
    ref = oracle.sweep(g, 19, 0, K, checks=False, sampler=sampler)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * K)
    G.set_sampler(sampler)
    for sched in (dict(), dict(path=2), dict(grid=1)):
        if sched and K > 500:
            continue
        G.set_schedule(**sched)
        G.cloud_reset()
        sw = G.sweep_range(0, K, 19, tree_switches=True).cpu().numpy().astype(np.uint64)
        assert np.array_equal(sw, ref.trees[:, 0]), sched
        assert np.array_equal(G.cloud(), ref.cloud), sched
    G.close()


def test_components_are_searched_side_by_side():
    # a chain is as long as its component: 16 of 1,000 vertices in less than
    # half the time of one of 16,000
    def ms(g):
        G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=64)
        G.set_sampler("rdfs")
        best = float("inf")
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            G.cloud_reset()
            a.record()
            G.sweep(8, 5)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        G.close()
        return best

    assert ms(_pieces([1000] * 16, 0)) < ms(_pieces([16000], 0)) / 2
