"""The windowed-lane kernels and the launch code that chooses them, run on the
host under AddressSanitizer (tests/windowed_host.cpp) and compared with the
oracle: lines that split into lanes of one size or of two, rings around a line
that no row count divides, lines in several chunks, odd and even numbers of
lines, padded rows, in-place calls, acyclic lines, bands that vary by row, partitions
and batches."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"

# r n axis d0 d1 pitch cyclic halfwidth precision in_place partitions batch
WINDOWED = """
1 30 0 5 3 0 1 2 0 0 0 0
1 61 0 5 3 0 1 2 0 0 0 0
1 100 0 7 3 0 1 2 0 0 0 0
1 150 0 3 2 1 1 0 0 1 0 0
1 243 0 5 1 0 1 3 0 0 0 0
2 613 0 3 2 0 1 3 0 0 0 0
1 701 0 2 2 3 1 2 0 0 0 0
1 928 0 2 1 0 1 2 0 0 0 0
1 929 0 2 1 0 1 2 0 0 0 0
2 1900 0 2 1 0 1 0 0 0 0 0
1 2055 0 1 2 0 1 2 0 0 0 1
1 56 1 17 3 0 1 2 0 0 0 0
1 57 1 16 2 1 1 2 0 0 0 0
1 64 2 5 7 0 1 3 0 0 0 0
2 24 1 3 3 2 1 2 0 0 0 0
2 300 2 33 2 0 1 0 0 1 0 0
2 241 1 9 2 0 1 3 0 0 0 0
2 613 1 6 1 0 1 3 0 0 0 1
1 613 1 1 3 0 1 0 0 0 0 0
1 512 2 2 2 0 0 0 0 0 0 0
2 613 2 5 1 1 0 0 0 1 0 0
1 1025 1 5 2 0 1 2 0 0 0 0
2 1700 2 3 3 0 1 3 0 0 0 0
1 1700 1 33 1 0 0 0 0 0 0 0
1 2048 0 2 2 0 1 0 0 0 4 0
2 2048 1 17 2 0 1 0 0 0 8 1
1 64 0 5 3 0 1 2 2 0 0 0
1 384 0 3 2 1 1 0 2 1 0 0
2 128 0 5 1 0 1 3 2 0 0 1
1 200 2 9 2 0 1 0 2 1 0 0
1 144 0 30 3 0 2 0 0 0 0 0
1 301 0 4 2 1 3 2 0 0 0 0
1 1000 0 3 1 1 3 3 0 0 0 0
2 72 0 23 1 0 3 3 0 0 0 0
2 300 0 5 3 1 2 0 0 1 0 0
2 256 0 5 1 0 3 2 2 0 0 0
3 139 0 4 2 0 2 0 0 0 0 0
1 130 1 5 3 1 2 0 0 0 0 0
2 40 2 3 7 0 3 3 0 0 0 0
2 256 1 33 2 0 2 0 0 1 0 0
3 300 2 5 2 0 3 2 0 0 0 0
0 32 0 5 3 0 1 2 0 0 0 0
0 33 0 7 2 1 1 3 0 0 0 0
0 48 0 3 3 0 1 2 0 0 0 0
0 1024 0 3 2 0 1 3 0 0 0 0
0 1025 0 3 2 1 1 1 0 0 0 0
0 2071 0 2 2 0 1 3 0 0 0 0
"""
# in place in several chunks, unit-stride acyclic lines, short ones with
# tridiagonal bands that vary by row, plain FP32: the general kernels
GENERAL = """
1 1700 1 4 2 0 1 0 0 1 0 0
1 1900 0 2 2 0 1 0 0 1 0 0
1 300 0 2 2 0 0 0 0 0 0 0
1 100 0 2 2 0 2 0 0 0 0 0
1 300 1 4 2 0 1 2 1 0 0 0
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++ in the ROCm installation")
    d = str(tmp_path_factory.mktemp("windowed"))
    src = [os.path.join(ROOT, "tests", "windowed_host.cpp")] + \
        [os.path.join(ROOT, "paper_2101_02286_amd", "csrc", f) for f in ("api.cpp", "plan.cpp")]
    jobs, objs = [], []
    for f in src:
        objs.append(os.path.join(d, os.path.basename(f) + ".o"))
        jobs.append(subprocess.Popen([CLANG, "-O1", "-g1", "-std=c++17", "-fsanitize=address,undefined",
                                      "-fno-sanitize=alignment,vptr,function", "-w",
                                      "-I" + os.path.join(ROOT, "tests", "host_hip"), "-c", f, "-o", objs[-1]]))
    oracle = os.path.join(d, "oracle.o")
    subprocess.check_call(["gcc", "-O2", "-c", os.path.join(ROOT, "oracle", "cb_oracle.c"), "-o", oracle])
    assert all(j.wait() == 0 for j in jobs)
    exe = os.path.join(d, "windowed")
    subprocess.check_call([CLANG, "-fsanitize=address,undefined", *objs, oracle, "-o", exe, "-lpthread", "-lm"])
    return exe


@pytest.mark.parametrize("cases,windowed", [(WINDOWED, True), (GENERAL, False)], ids=["windowed", "general"])
def test_windowed_kernels_on_the_host(driver, cases, windowed):
    r = subprocess.run([driver], input=cases, capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    lines = r.stdout.split("\n")[:-1]
    assert r.returncode == 0 and len(lines) == len(cases.split("\n")) - 2, r.stdout[-2000:] + r.stderr[-2000:]
    for ln in lines:
        assert ln.startswith("ok ") and ("windowed=1" in ln) == windowed, ln
