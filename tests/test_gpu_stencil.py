"""GPU parity of the standalone stencil's kernels at the edges of their tiles:
unit-stride lines around whole lanes and wavefronts, strided lines around 64
pairs and 8, 16 and 64 rows, lines shorter than the stencil, views on odd offsets
and permuted views."""
import numpy as np
import pytest
import torch

from paper_2101_02286_amd import cb, synth

pytestmark = pytest.mark.gpu

STENCILS = [(-2, [-0.1, -0.8, 0.05, 0.7, 0.15]), (-1, [-1.5, 0.25, 1.5, 0.5]), (-3, [-.02, -.15, -.7, .1, .7, .15, .02]),
            (1, [2.5]), (-3, [0.5, -0.5])]


def check(f, axis, lo, c):
    got = torch.full_like(f, float("nan"))
    cb.rhs_stencil(cb.Stencil(lo, c), f, axis, out=got)
    a = f.cpu().numpy()
    ref = sum(ck * np.roll(a, -(lo + k), 2 - axis) for k, ck in enumerate(c))
    bound = 2 * len(c) * 2.0 ** -53 * sum(map(abs, c)) * np.abs(a).max()  # both sums, one rounding a tap and side
    assert np.abs(got.cpu().numpy() - ref).max() <= bound


def shape_of(axis, n, other):
    s = list(other)
    s.insert(axis, n)
    return s[2], s[1], s[0]


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 9, 16, 17, 31, 32, 33, 48, 63, 64, 65, 129, 500, 1023, 1024, 1025, 1040, 2071])
def test_line_lengths(gpu, axis, n):
    for lo, c in STENCILS:
        check(synth.random_uniform(shape_of(axis, n, (37, 3)), seed=n).to(gpu), axis, lo, c)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("width", [1, 2, 16, 127, 128, 129, 257])
def test_widths(gpu, axis, width):
    for lo, c in STENCILS:
        check(synth.random_uniform(shape_of(axis, 70, (width, 5)), seed=width).to(gpu), axis, lo, c)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("perm", [(0, 1, 2), (0, 2, 1), (1, 0, 2), (2, 1, 0)])
def test_views(gpu, axis, perm):
    """Part of a larger array, its axes in any order: what surrounds it stays."""
    big = synth.random_uniform((43, 70, 54), seed=3).to(gpu)
    out = torch.full_like(big, 5.0)
    v = (slice(1, 41), slice(2, 68), slice(1, 52))
    lo, c = STENCILS[0]
    f = big[v].permute(perm)
    cb.rhs_stencil(cb.Stencil(lo, c), f, axis, out=out[v].permute(perm))
    a = f.cpu().numpy()
    ref = sum(ck * np.roll(a, -(lo + k), 2 - axis) for k, ck in enumerate(c))
    assert np.abs(out[v].permute(perm).cpu().numpy() - ref).max() <= 2 * len(c) * 2.0 ** -53 * sum(map(abs, c))
    out[v] = 5.0
    assert bool((out == 5.0).all())
