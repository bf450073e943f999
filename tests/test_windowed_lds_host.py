"""What the windowed-lane kernels read of LDS, on the host with LDS that holds NaN
until it is written (tests/windowed_lds_host.cpp): batches whose items have
workgroups of different sizes, in both forms, acyclic
lines, and rows of unlike scale."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++ in the ROCm installation")
    d = str(tmp_path_factory.mktemp("windowed_lds"))
    src = [os.path.join(ROOT, "tests", "windowed_lds_host.cpp")] + \
        [os.path.join(ROOT, "paper_2101_02286_amd", "csrc", f) for f in ("api.cpp", "plan.cpp")]
    jobs, objs = [], []
    for f in src:
        objs.append(os.path.join(d, os.path.basename(f) + ".o"))
        jobs.append(subprocess.Popen([CLANG, "-O1", "-std=c++17", "-w", "-I" + os.path.join(ROOT, "tests", "host_hip"),
                                      "-c", f, "-o", objs[-1]]))
    oracle = os.path.join(d, "oracle.o")
    subprocess.check_call(["gcc", "-O2", "-c", os.path.join(ROOT, "oracle", "cb_oracle.c"), "-o", oracle])
    assert all(j.wait() == 0 for j in jobs)
    exe = os.path.join(d, "windowed_lds")
    subprocess.check_call([CLANG, *objs, oracle, "-o", exe, "-lpthread", "-lm"])
    return exe


def run(driver, cases):
    """The driver's line for each case: all "ok"."""
    r = subprocess.run([driver], input="\n".join(cases) + "\n", capture_output=True, text=True, timeout=600)
    lines = r.stdout.split("\n")[:-1]
    assert r.returncode == 0 and len(lines) == len(cases), r.stdout[-3000:] + r.stderr[-3000:]
    for ln in lines:
        assert ln.startswith("ok "), ln
    return lines


# Launches, then r and n of the items.  Lanes of two sizes whose window table has
# more words than the item's workgroup has threads, beside a wider workgroup;
# lanes of one size (another instance, another launch); tables that fit.
MIXED = [(1, 2, 217, 613), (1, 2, 233, 500), (1, 2, 143, 613), (1, 2, 159, 613), (1, 3, 300, 613), (2, 2, 128, 613),
         (1, 2, 613, 217), (2, 2, 217, 613, 45), (1, 1, 401, 613)]


@pytest.mark.parametrize("form", [1, 2], ids=["per_tile", "queue"])
def test_batches_of_unlike_workgroups(driver, form):
    """One launch for the items of an instance, each item right, in both forms of a batch."""
    cases = ["%d %d " % (form, len(n)) + " ".join("%d %d %d %d 2 1 %d" % (r, m, 1 + form % 2, 5 + k, 3 * (k < 2))
                                                  for k, m in enumerate(n)) for _, r, *n in MIXED]
    for ln, case in zip(run(driver, cases), MIXED):
        assert "windowed=%d " % case[0] in ln, (case, ln)


# short acyclic lines, whose window would be wider than the line, and longer ones
ACYCLIC = [(1, 22), (1, 24), (1, 32), (1, 40), (1, 44), (1, 60), (2, 24), (2, 32), (2, 45), (2, 60), (2, 63),
           (2, 72), (2, 100), (3, 48), (3, 288)]


@pytest.mark.parametrize("axis", [1, 2])
def test_acyclic_lines(driver, axis):
    """Single calls, and pairs of such lines in one batch: each on a windowed kernel."""
    lines = run(driver, ["0 1 %d %d %d 9 3 0 0" % (r, n, axis) for r, n in ACYCLIC])
    assert all("windowed=1 " in ln for ln in lines)
    run(driver, ["1 2 %d %d %d 9 3 0 0 %d %d %d 5 2 0 0" % (r, n, axis, r, n, axis) for r, n in ACYCLIC])


@pytest.mark.parametrize("n", [39, 44, 66, 88, 128, 130, 200])
def test_rows_of_unlike_scale(driver, n):
    """Per-row bands, half of them scaled with their right-hand side: as exact as without."""
    lines = run(driver, ["0 1 1 %d %d 5 2 %d 0" % (n, axis, c) for axis in (1, 2) for c in (2, 3)])
    assert any("windowed=1 " in ln for ln in lines)
