"""A batch's trees in LDS at the sizes where they stop fitting, and tree counts
around an item's, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")

SETS = {
    "small": lambda: [synth.isolated_vertices(5), synth.random_tree(2, 1), synth.random_small(300, 250, 2, p_pos=0.5),
                      synth.cycle_graph(33, (0,)), synth.erdos_renyi_connected(300, 32 * 256 + 1, 0.8, 3),
                      synth.erdos_renyi_connected(2048, 5000, 0.8, 4)],
    "blocks": lambda: [synth.erdos_renyi_connected(n, 2 * n, 0.8, n) for n in (2049, 7500, 7501, 40)],
    "lds_most": lambda: [synth.erdos_renyi_connected(n, 2 * n, 0.8, n) for n in (15000, 90)],
    "lds_over": lambda: [synth.erdos_renyi_connected(n, 2 * n, 0.8, n) for n in (15001, 15000, 90)],
}


@pytest.mark.parametrize("name", SETS)
@pytest.mark.parametrize("K", [1, 15, 40])
def test_batch_edges_matches_oracle(name, K):
    graphs = SETS[name]()
    ref = [oracle.sweep(g, 31, 0, K, checks=False) for g in graphs]
    B = fr.BatchGraph(graphs, cloud_capacity_per_graph=K)
    for path, block, grid in ((0, 256, 0), (1, 256, 1), (1, 512, 0), (1, 1024, 2)):
        B.set_schedule(path=path, block=block, grid=grid)
        least, distinct = B.sweep(K, 31)
        for i, r in enumerate(ref):
            assert tuple(least[i].tolist()) == r.best, (path, block, i)
            assert np.array_equal(B.cloud(i), r.cloud), (path, block, i)
            assert int(distinct[i]) == len(r.cloud)
    B.close()
