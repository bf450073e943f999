"""Batches whose large items, or items alone in their kernel class, get launches of
their own: with a workgroup per tile, with the persistent queue and replayed
from a graph, against single calls, bit for bit."""
import pytest
import torch

from oracle import schemes
from paper_2101_02286_amd import cb, synth

pytestmark = pytest.mark.gpu

TRI = schemes.bands_collocated(schemes.DERIV6)
# (nz, ny, nx): 2^24 points and one line more or less beside smaller ones
SHAPES = [(256, 256, 256), (256, 255, 256), (257, 256, 256), (256, 30, 40), (20, 256, 30), (9, 11, 256)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_own_launches(gpu, precision):
    plan = cb.Plan(TRI, 256, precision=precision)
    st = cb.Stencil(-2, [-0.1, -0.8, 0.05, 0.7, 0.15])
    items, singles = [], []
    for k, shape in enumerate(SHAPES):
        f = synth.random_uniform(shape, seed=k).to(gpu)
        for axis in range(3):
            if shape[2 - axis] == 256:
                items.append((plan, st, f, torch.empty_like(f), axis))
                singles.append(cb.apply_derivative(plan, st, f, axis))
    batch = cb.Batch(items)
    graph = torch.cuda.CUDAGraph()
    batch.launch()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        batch.launch()
    for run in (batch.launch, lambda: batch.launch(max_ctas=13), graph.replay, graph.replay):
        for it in items:
            it[3].fill_(float("nan"))
        run()
        torch.cuda.synchronize()
        for it, single in zip(items, singles):
            assert torch.equal(it[3], single)
