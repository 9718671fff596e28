"""The descent reads a plain Gamma_0 where it lies; every other one is copied
first, so what a copy would have resolved is kept."""
import pytest
import torch

from paper_2311_00869_amd import synth

pytestmark = pytest.mark.gpu

fr = pytest.importorskip("paper_2311_00869_amd.frustration")


@pytest.fixture(scope="module")
def graph():
    # two hubs with rows of several items, and short rows
    g = synth.chung_lu(6000, 24000, 2.1, 3, p_pos=0.8)
    G = fr.Graph(g.row_ptr, g.col, g.sign, cloud_capacity=4)
    yield G
    G.close()


def _start(G, R=8):
    return torch.from_numpy(synth.graphl_init(G.n, R, 5)).cuda()


@pytest.mark.parametrize("steps", [0, 3])
def test_start_that_is_a_lazy_negation(graph, steps):
    gamma = _start(graph)
    lazy = torch._neg_view(gamma)
    assert lazy.is_neg() and lazy.is_contiguous()
    want, _ = graph.graphl_descend(-gamma, steps)
    got, _ = graph.graphl_descend(lazy, steps)
    assert torch.equal(got, want)


@pytest.mark.parametrize("steps", [0, 3])
def test_start_with_a_forward_tangent(graph, steps):
    import torch.autograd.forward_ad as ad
    gamma = _start(graph)
    tangent = torch.ones_like(gamma)
    want, _ = graph.graphl_descend(gamma, steps)
    with ad.dual_level():
        got, _ = graph.graphl_descend(ad.make_dual(gamma, tangent), steps)
        primal, kept = ad.unpack_dual(got)
        assert torch.equal(primal, want) and kept is not None and torch.equal(kept, tangent)


@pytest.mark.parametrize("R", [4, 32])
def test_start_off_the_vector_alignment(graph, R):
    # rows of several items are summed by the lane layout, which the alignment
    # chooses: a start off it gives the same bits as one on it
    gamma = _start(graph, R)
    flat = torch.empty(gamma.numel() + 1, device="cuda")
    shifted = flat[1:].view(gamma.shape)
    shifted.copy_(gamma)
    assert shifted.data_ptr() % 16 and shifted.is_contiguous()
    want, _ = graph.graphl_descend(gamma, 3)
    got, _ = graph.graphl_descend(shifted, 3)
    assert torch.equal(got, want)
