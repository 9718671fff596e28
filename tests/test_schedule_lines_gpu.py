"""Where the automatic schedule of a graph whose trees fit LDS turns to the
multi-tree path: 65,536 edges, and 80 million edges times trees.  The phase log
tells which ran; whole numbers, so equal to the oracle."""
import numpy as np
import pytest

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


@pytest.mark.parametrize("m,trees,multi", [(65535, 1221, False), (65536, 1220, False), (65536, 1221, True),
                                           (100000, 799, False), (100000, 800, True)])
def test_either_side_of_the_lines(m, trees, multi):
    g = synth.erdos_renyi_connected(2500, m, 0.8, 8)
    seed = 3
    ref = oracle.sweep(g, seed, 0, trees, checks=False)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=2 * trees)
    for log in (4096, 0):
        buf = G.phase_log(log)
        G.cloud_reset()
        sw = G.sweep_range(0, trees, seed, tree_switches=True).cpu().numpy().astype(np.uint64)
        if log:
            assert (int(buf[0]) > 0) == multi
        assert np.array_equal(sw, ref.trees[:, 0])
        assert np.array_equal(G.cloud(), ref.cloud)
    G.close()
