"""A NaN or infinity in the input stays in its own line, on lanes that share a
wavefront, a pair or an LDS plane with others', and shows around its row."""
import pytest
import torch

from oracle import schemes
from paper_2101_02286_amd import cb, synth

pytestmark = pytest.mark.gpu

BANDS = dict(tri=schemes.bands_collocated(schemes.DERIV6), penta=schemes.bands_collocated(schemes.DERIV10))


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("band,per_row", [("tri", False), ("penta", False), ("penta", True)])
@pytest.mark.parametrize("n", [64, 97, 300, 613, 1100])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_other_lines(gpu, axis, band, per_row, n, value):
    shape = [9, 37]
    shape.insert(2 - axis, n)
    b = synth.random_uniform(tuple(shape), seed=n).to(gpu)
    bands = synth.random_bands(n, 2, seed=n) if per_row else BANDS[band]
    plan = cb.Plan(bands, n, per_row=per_row)
    want = cb.solve(plan, b, axis)
    lines = b.movedim(2 - axis, -1)  # (9, 37, n)
    at = [(4, 18, n // 2), (0, 0, 0), (8, 36, n - 1)]
    for u, v, j in at:
        lines[u, v, j] = value
    got = cb.solve(plan, b, axis).movedim(2 - axis, -1)
    want = want.movedim(2 - axis, -1).clone()
    for u, v, j in at:
        assert not torch.isfinite(got[u, v, j])
        got[u, v], want[u, v] = 0.0, 0.0
    assert torch.equal(got, want)
