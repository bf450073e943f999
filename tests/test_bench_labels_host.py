"""The bench names the kernel instances that its launches run, from the plan's layouts."""
import pytest

import bench
from paper_2101_02286_amd import cb, schemes


def instances(path):
    import os
    import re
    csrc = os.path.join(os.path.dirname(cb.__file__), "csrc")
    return re.findall(r"CB_WIN_([XS])\((\d), (\d+)\)", open(os.path.join(csrc, path)).read())


@pytest.mark.parametrize("n", [64, 256, 500, 512, 613, 2500, 8192])
@pytest.mark.parametrize("scheme", ["tri6", "penta10", "hept12"])
def test_labels(scheme, n):
    plan = cb.Plan(schemes.bands(scheme), n, host_only=True)
    r = plan.r
    for axis in range(3):
        label, rows = bench.kernel_group(plan, axis), bench.windowed_rows(plan, axis)
        assert label.startswith("k_win " if rows else "k_line ")
        assert ("/r%d/rows" % r) in label and (axis == 0) == ("unit-stride" in label)
        if rows:  # an instance that exists
            kind = "X" if axis == 0 else "S"
            assert (kind, str(r), str(rows)) in instances("win_r%d_%s.hip" % (r, kind.lower()))
    plan.close()


def test_headline_labels():
    plan = cb.Plan(schemes.bands("tri6"), 512, host_only=True)
    assert bench.kernel_group(plan, 0) == "k_line unit-stride/r1/rows8/pcr"
    assert bench.kernel_group(plan, 1) == bench.kernel_group(plan, 2) == "k_win strided/r1/rows16"
    plan.close()
    plan = cb.Plan(schemes.bands("tri6"), 512, rows_per_lane=32, interior=2, host_only=True)
    assert bench.kernel_group(plan, 1) == "k_line strided/r1/rows32/elim"
    plan.close()


def test_window_array():
    plan = cb.Plan(schemes.bands("tri6"), 512, host_only=True)
    assert list(plan.array(13, 0)) == [] and list(plan.array(13, 1)) == [16, 32, 16, 0, 2, 0]
    with pytest.raises(cb.CbError):
        plan.array(13, 2)
    with pytest.raises(cb.CbError):
        plan.array(14)
    plan.close()


@pytest.mark.parametrize("scheme,count", [("tri6", 1), ("penta10", 2)])
def test_refinements(scheme, count):
    """Refinement iterations as the launches run them: none where they solve in FP64."""
    bands = schemes.bands(scheme)
    plan = cb.Plan(bands, 500, precision="fp32_refine", host_only=True)
    assert plan.info()["refine_iters"] == count and [bench.refinements(plan, ax) for ax in range(3)] == [0, 0, 0]
    plan.close()
    plan = cb.Plan(bands, 512, precision="fp32_refine", rows_per_lane=8, host_only=True)
    assert [bench.refinements(plan, ax) for ax in range(3)] == [count] * 3
    plan.close()
    plan = cb.Plan(bands, 512, host_only=True)
    assert bench.refinements(plan, 1) == 0
    plan.close()
