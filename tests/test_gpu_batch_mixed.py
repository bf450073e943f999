"""Batches of strided items of one kernel instance with workgroups of different
sizes, lanes of two sizes among them: in either form against single calls and
the oracle."""
import numpy as np
import pytest
import torch

import oracle
from oracle import schemes
from paper_2101_02286_amd import cb, synth

pytestmark = pytest.mark.gpu

BANDS = dict(tri=schemes.bands_collocated(schemes.DERIV6), penta=schemes.bands_collocated(schemes.DERIV10),
             hept=schemes.bands_collocated(schemes.DERIV12H))
LO, C = -3, [-.02, -.15, -.7, .1, .7, .15, .02]
TOL = 1e-12  # the library's FP64 bound against the oracle


@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("band,ns", [("penta", (125, 613, 126, 500, 143, 159, 45)), ("hept", (250, 500, 157, 333)),
                                     ("tri", (401, 613, 257, 57, 431))])
def test_unlike_workgroups(gpu, axis, band, ns):
    st = cb.Stencil(LO, C)
    items, singles, refs = [], [], []
    for k, n in enumerate(ns):
        shape = (3, n, 37 + k) if axis == 1 else (n, 3, 37 + k)
        f = synth.random_uniform(shape, seed=n)
        plan = cb.Plan(BANDS[band], n)
        items.append((plan, st, f.to(gpu), torch.empty(shape, dtype=torch.float64, device=gpu), axis))
        singles.append(cb.apply_derivative(plan, st, items[-1][2], axis))
        refs.append(oracle.apply_axis(f.numpy(), axis, BANDS[band], LO, C))
    batch = cb.Batch(items)
    for max_ctas in (-1, 0, 3):
        for it in items:
            it[3].fill_(float("nan"))
        batch.launch(max_ctas=max_ctas)
        torch.cuda.synchronize()
        for it, single, ref in zip(items, singles, refs):
            assert torch.equal(it[3], single)
            assert np.abs(it[3].cpu().numpy() - ref).max() <= TOL * np.abs(ref).max()
