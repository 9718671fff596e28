"""What a NaN in Gamma does to the overflow policy's scales, for each route of
the descent: it is above every threshold, except in the main component of
graphs with long rows or of more than 4,096 vertices, where it is passed over."""
import numpy as np
import pytest
import torch

from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


def _with_pairs(g, pairs):
    """g, the main component, and pairs of vertices beside it."""
    u = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    up = u < g.col
    a = g.n + 2 * np.arange(pairs)
    return synth.csr_from_edges(g.n + 2 * pairs, np.concatenate([u[up], a]), np.concatenate([g.col[up], a + 1]),
                                np.concatenate([g.sign[up], np.ones(pairs, np.int64)]))


# main component, and whether a NaN counts there: one launch without and with
# long rows, a launch per step for many entries or many vertices
GRAPHS = {
    "small": (lambda: synth.erdos_renyi_connected(500, 2000, 0.8, 1), True),
    "small_long_rows": (lambda: synth.chung_lu(3000, 12000, 2.1, 3, p_pos=0.8), False),
    "many_entries": (lambda: synth.erdos_renyi_connected(2000, 70000, 0.8, 2), True),
    "many_entries_long_rows": (lambda: synth.erdos_renyi_connected(1000, 150000, 0.8, 2), False),
    "many_vertices": (lambda: synth.erdos_renyi_connected(5000, 20000, 0.8, 4), False),
}


@pytest.mark.parametrize("name", GRAPHS)
@pytest.mark.parametrize("R", [3, 8])
def test_scales_beside_a_nan(name, R):
    make, counts = GRAPHS[name]
    g = make()
    hub = int(np.argmax(np.diff(g.row_ptr)))
    n, steps, shift = g.n, 6, 40
    g = _with_pairs(g, 3)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    gamma = torch.from_numpy(synth.graphl_init(g.n, R, 5)).cuda()
    gamma[hub, 0] = float("nan")   # the main component of restart 0
    gamma[n + 2, 1] = float("nan")  # a pair of restart 1
    out, scales = G.graphl_descend(gamma, steps, 0.001, rescale_log2=shift)
    s = scales().cpu().numpy()
    # each step after the first reads it; nothing else comes near the threshold
    every = shift * (steps - 1)
    want = np.zeros((g.n, R), np.int32)
    want[n + 2:n + 4, 1] = every
    if counts:
        main = np.zeros(g.n, bool)
        main[:n] = np.diff(g.row_ptr)[:n] > 0
        main &= s[:, 0] != 0  # (vertices of other small components of the generator stay at 0)
        assert main[hub] and main.sum() > n // 2
        want[main, 0] = every
    assert np.array_equal(s, want)
    assert torch.isnan(out[hub, 0]) and torch.isnan(out[n + 2:n + 4, 1]).all()
    assert torch.isfinite(out[:, 2]).all()
    G.close()
