"""Which plans get windowed lanes, and how wide their windows are, does not depend on
the scale of the bands or of single rows: what bounds the growth of an elimination
and what a window may leave out is measured beside the rows' own entries."""
import numpy as np
import pytest

from paper_2101_02286_amd import cb, schemes, synth

# the schemes, and bands whose elimination grows by 2^8 and more within a lane
BANDS = [schemes.bands("tri6"), schemes.bands("penta10"), schemes.bands("hept12"), [1.5, 1.0, 0.2], [2.0, 1.0, 0.05],
         [3.0, 1.0, 0.01], [0.3, 1.6, 1.0, 0.1, 0.02]]


def layouts(bands, n, **kw):
    plan = cb.Plan(bands, n, host_only=True, **kw)
    out = [list(plan.array(13, s)) for s in (0, 1)]
    plan.close()
    return out


@pytest.mark.parametrize("cyclic", [True, False])
@pytest.mark.parametrize("bands", BANDS, ids=lambda b: "%g,%g" % (b[0], b[1]))
def test_scaled_bands(bands, cyclic):
    for n in (24, 40, 60, 149, 300, 613):
        for e in (-40, -13, -3, 3, 13, 40):
            try:
                got, want = [layouts(b, n, cyclic=cyclic) for b in (np.ldexp(bands, e), bands)]
            except cb.CbError:  # no plan, and no layout
                continue
            assert got == want, (n, e)


def test_growth_needs_pivoting():
    """An elimination that grows by 1.5^10 within a lane stays with the general kernels."""
    for e in (-40, -13, 0, 13):
        assert layouts(np.ldexp([1.5, 1.0, 0.2], e), 149)[1] == []


@pytest.mark.parametrize("cyclic", [True, False])
@pytest.mark.parametrize("r", [1, 2, 3])
def test_scaled_rows(r, cyclic):
    same = 0
    for n in (40, 66, 130, 200, 300):
        bands = np.asarray(synth.random_bands(n, r, seed=n))
        want = layouts(bands, n, cyclic=cyclic, per_row=True)
        for rows in (slice(0, n // 2), slice(0, 1), slice(0, n, 3)):
            for e in (-9, 9):
                scaled = bands.copy()
                scaled[rows] = np.ldexp(scaled[rows], e)
                for got, w in zip(layouts(scaled, n, cyclic=cyclic, per_row=True), want):
                    if got and w and got[0] == w[0]:  # (a layout may be refused, not chosen otherwise)
                        assert got == w, (n, rows, e)
                        same += 1
    assert same > 10
