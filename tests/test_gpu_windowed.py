"""GPU parity of the windowed-lane launches at the edges of their layouts: line
lengths around whole lanes, whole wavefronts and whole workgroups, lanes of one
size and of two, odd numbers of adjacent lines, rows that start on any 8-byte
address, one chunk more or less."""
import numpy as np
import pytest
import torch

import oracle
from oracle import schemes
from paper_2101_02286_amd import cb, synth

pytestmark = pytest.mark.gpu

BANDS = dict(tri=schemes.bands_collocated(schemes.DERIV6), penta=schemes.bands_collocated(schemes.DERIV10),
             hept=schemes.bands_collocated(schemes.DERIV12H))
STENCILS = dict(tri=(-2, [-0.1, -0.8, 0.05, 0.7, 0.15]), penta=(-3, [-.02, -.15, -.7, .1, .7, .15, .02]),
                hept=(-3, [-.02, -.15, -.7, .1, .7, .15, .02]))
TOL = 1e-12  # the library's FP64 bound against the oracle


def relerr(x, ref):
    return float(np.abs(x - ref).max() / np.abs(ref).max())


def grid(axis, n, other):
    s = list(other)
    s.insert(axis, n)
    return s[2], s[1], s[0]  # (nz, ny, nx)


# unit-stride: the shortest ring, exact splits, a wavefront's last lane (928 =
# 58 x 16 rows and 6 halo lanes), chunks; strided: 32 and 64 lanes, chunks
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("band", ["tri", "penta", "hept"])
@pytest.mark.parametrize("n", [57, 100, 145, 255, 257, 383, 511, 513, 640, 927, 929, 1023, 1025, 1857, 2049, 4111])
def test_line_lengths(gpu, axis, band, n):
    shape = grid(axis, n, (37, 3))
    f = synth.random_uniform(shape, seed=n)
    lo, c = STENCILS[band]
    plan = cb.Plan(BANDS[band], n)
    out = torch.full(shape, float("nan"), dtype=torch.float64, device=gpu)
    cb.apply_derivative(plan, cb.Stencil(lo, c), f.to(gpu), axis, out=out)
    assert relerr(out.cpu().numpy(), oracle.apply_axis(f.numpy(), axis, BANDS[band], lo, c)) <= TOL
    ref = oracle.solve_axis(f.numpy(), axis, BANDS[band])
    assert relerr(cb.solve(plan, f.to(gpu), axis).cpu().numpy(), ref) <= TOL
    x = f.to(gpu)
    cb.solve(plan, x, axis, out=x)  # in place
    assert relerr(x.cpu().numpy(), ref) <= TOL


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("n", [500, 613])
@pytest.mark.parametrize("width", [1, 2, 31, 33, 64])
def test_views(gpu, axis, n, width):
    """Rows inside a larger array at odd offsets: aligned and unaligned, lines
    in runs across planes and not; what surrounds them stays as it was."""
    shape = grid(axis, n, (width, 3))
    big = synth.random_uniform(tuple(s + 3 for s in shape), seed=width).to(gpu)
    before = big.clone()
    for off in (0, 1):
        v = tuple(slice(off, off + s) for s in shape)
        out = torch.full_like(big, 5.0)
        cb.solve(cb.Plan(BANDS["tri"], n), big[v], axis, out=out[v])
        ref = oracle.solve_axis(np.ascontiguousarray(big[v].cpu().numpy()), axis, BANDS["tri"])
        assert relerr(out[v].cpu().numpy(), ref) <= TOL
        out[v] = 5.0
        assert bool((out == 5.0).all()) and torch.equal(big, before)


@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("band", ["tri", "penta"])
@pytest.mark.parametrize("n", [60, 200, 301, 512, 900, 1100])
def test_acyclic_strided(gpu, axis, band, n):
    b = synth.random_uniform(grid(axis, n, (19, 2)), seed=n)
    x = cb.solve(cb.Plan(BANDS[band], n, cyclic=False), b.to(gpu), axis).cpu().numpy()
    assert relerr(x, oracle.solve_axis(b.numpy(), axis, BANDS[band], cyclic=False)) <= TOL


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("n,P", [(2048, 4), (4000, 8), (8192, 16), (7680, 15)])
def test_partitions(gpu, axis, n, P):
    b = synth.random_uniform(grid(axis, n, (17, 2)), seed=P)
    for band in ("tri", "penta"):
        x = cb.solve(cb.Plan(BANDS[band], n, partitions=P), b.to(gpu), axis).cpu().numpy()
        assert relerr(x, oracle.solve_axis(b.numpy(), axis, BANDS[band])) <= TOL


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("band", ["tri", "penta", "hept"])
@pytest.mark.parametrize("n", [64, 96, 128, 192, 320, 384, 512, 613, 1024, 2048])
def test_refined_plans(gpu, axis, band, n):
    """FP32 + refinement: solves to the FP64 bound, whatever count is asked for."""
    shape = grid(axis, n, (35, 3))
    f = synth.random_uniform(shape, seed=n)
    lo, c = STENCILS[band]
    ref = oracle.apply_axis(f.numpy(), axis, BANDS[band], lo, c)
    for iters in (0, 3):
        plan = cb.Plan(BANDS[band], n, precision="fp32_refine", refine_iters=iters)
        x = cb.apply_derivative(plan, cb.Stencil(lo, c), f.to(gpu), axis).cpu().numpy()
        assert relerr(x, ref) <= TOL


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("r", [1, 2, 3])
@pytest.mark.parametrize("cyclic", [True, False])
@pytest.mark.parametrize("n", [24, 41, 64, 100, 129, 250, 300, 512, 613, 701, 1000])
def test_bands_by_row(gpu, axis, r, cyclic, n):
    """Lanes with coefficients of their own, odd numbers of lines, in place."""
    shape = grid(axis, n, (35, 3))
    bands = synth.random_bands(n, r, seed=n)
    b = synth.random_uniform(shape, seed=n + r)
    ref = oracle.solve_axis(b.numpy(), axis, bands, cyclic=cyclic, per_row=True)
    plan = cb.Plan(bands, n, cyclic=cyclic, per_row=True)
    x = b.to(gpu)
    assert relerr(cb.solve(plan, x, axis).cpu().numpy(), ref) <= TOL
    cb.solve(plan, x, axis, out=x)
    assert relerr(x.cpu().numpy(), ref) <= TOL
    if cyclic:
        lo, c = STENCILS["tri" if r == 1 else "penta"]
        x = cb.apply_derivative(plan, cb.Stencil(lo, c), b.to(gpu), axis).cpu().numpy()
        rhs = sum(ck * np.roll(b.numpy(), -(lo + k), 2 - axis) for k, ck in enumerate(c))
        assert relerr(x, oracle.solve_axis(rhs, axis, bands, per_row=True)) <= TOL
