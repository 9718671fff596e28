"""The one-launch descent of a small graph at the edges of its row counts, held
entries and long rows, against the float64 oracle and against itself step by
step."""
import numpy as np
import pytest
import torch

from oracle import graphl as ogl
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

ALPHA = 0.01


def _hubs(n):
    """Rows of 7 .. 700 entries over a cycle, a second component and vertices
    without edges."""
    rng = np.random.default_rng(n)
    deg = (7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 40, 41, 255, 256, 257, 300, 513, 700)
    pool = n - len(deg) - 8
    us = [np.arange(pool), np.array([n - 5, n - 4])] + [np.full(d, pool + i) for i, d in enumerate(deg)]
    vs = [(np.arange(pool) + 1) % pool, np.array([n - 4, n - 3])] + [rng.choice(pool, d, replace=False) for d in deg]
    u, v = np.concatenate(us), np.concatenate(vs)
    return synth.csr_from_edges(n, u, v, np.where(rng.random(u.size) < 0.6, 1, -1))


GRAPHS = {
    "pair": lambda: synth.cycle_graph(3, (0,)),
    "1023": lambda: synth.erdos_renyi_connected(1023, 5000, 0.8, 1),
    "1024_dense": lambda: synth.erdos_renyi_connected(1024, 20000, 0.8, 2),
    "1025": lambda: synth.erdos_renyi_connected(1025, 5000, 0.8, 3),
    "2048_dense": lambda: synth.erdos_renyi_connected(2048, 30000, 0.8, 4),
    "2049": lambda: synth.erdos_renyi_connected(2049, 30000, 0.8, 5),
    "4096": lambda: synth.erdos_renyi_connected(4096, 50000, 0.8, 6),
    "4097": lambda: synth.erdos_renyi_connected(4097, 50000, 0.8, 7),
    "entries_most": lambda: synth.erdos_renyi_connected(1500, 65536, 0.8, 8),
    "entries_over": lambda: synth.erdos_renyi_connected(1500, 65537, 0.8, 8),
    "hubs1024": lambda: _hubs(1024),
    "hubs1500": lambda: _hubs(1500),
    "hubs4096": lambda: _hubs(4096),
    "components": lambda: synth.random_small(3000, 2500, 6, p_pos=0.6),
    "edgeless": lambda: synth.isolated_vertices(70),
}


@pytest.mark.parametrize("name", GRAPHS)
@pytest.mark.parametrize("R", [1, 5, 32])
def test_small_descent(name, R):
    from paper_2311_00869_amd import frustration as fr
    g = GRAPHS[name]()
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    gamma = torch.from_numpy(synth.graphl_init(g.n, R, 5)).cuda()
    x = gamma.cpu().numpy()
    one, scales = G.graphl_descend(gamma, 1, ALPHA)
    want = x.astype(np.float64) - ALPHA * ogl.grad(g, x)
    # each row: d adds and the update, each off by half an ulp of a partial
    # result of at most the sum of magnitudes
    deg = np.diff(g.row_ptr).astype(np.float64)
    mag = np.zeros(x.shape)
    np.add.at(mag, np.repeat(np.arange(g.n), np.diff(g.row_ptr)), np.abs(x[g.col]))
    bound = (deg[:, None] + 8) * 2.0**-24 * (np.abs(x) + ALPHA * mag)
    assert np.all(np.abs(one.cpu().numpy() - want) <= bound)
    assert not scales().any()
    # several steps are the steps one by one
    step = gamma
    for k in range(1, 6):
        step, _ = G.graphl_descend(step, 1, ALPHA)
        several, _ = G.graphl_descend(gamma, k, ALPHA)
        assert torch.equal(several, step), k
    G.close()


@pytest.mark.parametrize("n", [1024, 2000, 4096])
def test_small_descent_with_hubs_is_exact_across_rescaling(n):
    from paper_2311_00869_amd import frustration as fr
    g = _hubs(n)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    gamma = torch.from_numpy(synth.graphl_init(g.n, 5, 12)).cuda()
    a, sa = G.graphl_descend(gamma, 150, 0.2, rescale_log2=8)
    b, sb = G.graphl_descend(gamma, 150, 0.2, rescale_log2=64)
    assert torch.isfinite(a).all() and int(sa().max()) >= 128
    ta = np.ldexp(a.cpu().numpy().astype(np.float64), sa().cpu().numpy())
    tb = np.ldexp(b.cpu().numpy().astype(np.float64), sb().cpu().numpy())
    assert np.array_equal(ta, tb)
    G.close()
