"""Plans with lanes of their own coefficients: the inverse of their reduced system,
and no tables for launches that would not use them."""
import os
import re
import subprocess

import pytest

from paper_2101_02286_amd import cb, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_inverses_of_the_reduced_system(tmp_path):
    exe = str(tmp_path / "window_inverse")
    subprocess.check_call(["g++", "-O1", "-std=c++17", os.path.join(ROOT, "tests", "window_inverse.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True).stdout
    kept, lost = map(int, re.search(r"^ok kept (\d+) lost (\d+)$", out, re.M).groups())
    assert kept > 300 and lost > 20, out


@pytest.mark.parametrize("r,n,unit_stride", [(1, 300, True), (2, 300, True), (3, 300, True), (1, 1000, True),
                                             (3, 1000, False), (3, 800, False)])
def test_tables_that_fit(r, n, unit_stride):
    """Unit-stride launches take lanes of their own coefficients where a compute unit holds four wavefronts of them."""
    plan = cb.Plan(synth.random_bands(n, r, seed=1), n, per_row=True, host_only=True)
    assert (len(plan.array(13, 0)) > 0) == unit_stride and len(plan.array(13, 1)) > 0
    plan.close()
