"""The descent of graphs of many components: as fast as of one, and the same
true iterate whatever the threshold of the scales."""
import numpy as np
import pytest
import torch

from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _rings(count, size, chords=0):
    a = np.arange(count * size)
    u, v = [a], [a - a % size + (a + 1) % size]
    if chords:  # every tenth vertex of a ring to its first: rows of up to `chords`
        x = a[(a % size > 1) & (a % size < size - 1)][:: max(1, size // chords)]
        u.append(x)
        v.append(x - x % size)
    u, v = np.concatenate(u), np.concatenate(v)
    return synth.csr_from_edges(count * size, u, v, np.where(np.random.default_rng(1).random(u.size) < 0.7, 1, -1))


def _step_us(g, R):
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    gamma = torch.from_numpy(synth.graphl_init(g.n, R, 5)).cuda()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        G.graphl_descend(gamma, 40)
        b.record()
        torch.cuda.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b) / 40)
    G.close()
    return best


@pytest.mark.parametrize("R", [16, 64])
def test_many_components_cost_no_more_than_one(R):
    assert _step_us(_rings(20, 1000), R) <= 2 * _step_us(_rings(1, 20000), R)


@pytest.mark.parametrize("R", [3, 32])
def test_components_rescale_exactly(R):
    # hubs of 90 entries in every component, so that the iterates grow past 2^8
    # every few steps; beside them components that do not grow
    g = _rings(12, 900, 90)
    pad = 6000
    u = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    up = u < g.col
    a = g.n + 2 * np.arange(pad // 2)
    g = synth.csr_from_edges(g.n + pad, np.concatenate([u[up], a]), np.concatenate([g.col[up], a + 1]),
                             np.concatenate([g.sign[up], np.ones(a.size, np.int64)]))
    assert g.n > 4096
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    gamma = torch.from_numpy(synth.graphl_init(g.n, R, 12)).cuda()
    true = []
    for shift in (8, 64):
        x, scales = G.graphl_descend(gamma, 60, 0.3, rescale_log2=shift)
        s = scales().cpu().numpy()
        assert torch.isfinite(x).all() and (shift == 64 or (s[: 12 * 900].max() >= 24 and s[-pad:].min() == 0))
        true.append(np.ldexp(x.cpu().numpy().astype(np.float64), s))
    assert np.array_equal(true[0], true[1])
    G.close()
