"""Launch shapes on a device of 256 compute units, by the library's launch code on
the host: strided lines that form one run across planes are tiled alike however
many of them lie in a plane; batches on the persistent queue."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
DRIVER = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <vector>
#include "launch.h"
namespace cb {
static const void *const kFn = (const void *)(uintptr_t)100;
const LineKernel *find_line_kernel(int, int, int, int, int, bool, bool) { return nullptr; }
const LineKernel *find_copy_kernel(int, int, bool) { return nullptr; }
const BatchKernel *find_batch_kernel(int, int, int, bool, bool, int, int) { return nullptr; }
const WgKernel *find_wg_kernel(int, int, int, int, bool) { return nullptr; }
const WgKernel *find_wg32_kernel(int, int, int, int, bool) { return nullptr; }
const WinKernel *find_win_kernel(int R, int M, int mode, int Q, bool uni) {
  static WinKernel k;
  k = WinKernel{R, M, mode, Q, uni, 1024, 8 * R, kFn, kFn};
  return &k;
}
const WinKernel *find_win_rows_kernel(int, int, int, int) { return nullptr; }
const WinKernel *find_win_copy_kernel(int, int, bool) { return nullptr; }
const void *stencil_kernel(int) { return nullptr; }
const WinKernel *find_win_stencil_kernel(int) { return nullptr; }
}  // namespace cb
hipError_t hipLaunchKernel(const void *, dim3 grid, dim3 block, void **, size_t, hipStream_t) {
  printf("%u x %u\n", grid.x, block.x);
  return hipSuccess;
}
int main() {
  const double bands[3] = {1 / 3., 1, 1 / 3.};
  long n, nx, ny;
  int batch;
  while (scanf("%ld %ld %ld %d", &n, &nx, &ny, &batch) == 4) {
    cb_plan_desc d = {};
    d.r = 1;
    d.n = (int)n;
    d.bands = bands;
    d.cyclic = 1;
    cb_plan_t p;
    if (cb_plan(&d, &p)) return 1;
    cb_grid g = {{nx, ny, n}, {1, nx, nx * ny}};
    const uintptr_t base = uintptr_t(1) << 40;
    cb_stencil st = {-2, 2, {1, 2, 0, 2, 1}};
    cb_batch_item it = {p, &st, g, 2, (double *)base, (double *)(2 * base)};
    std::vector<char> ws(cb_batch_workspace_bytes(&it, 1));
    if (batch ? cb_solve_batched(&it, 1, ws.data(), ws.size(), batch == 1 ? 0 : 64, nullptr)
              : cb_solve(p, &g, 2, (double *)base, (double *)(2 * base), nullptr))
      return 1;
    cb_plan_destroy(p);
  }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++ in the ROCm installation")
    d = tmp_path_factory.mktemp("shapes")
    csrc, host = os.path.join(ROOT, "paper_2101_02286_amd", "csrc"), os.path.join(ROOT, "tests", "host_hip")
    (d / "hip").mkdir()
    with open(os.path.join(host, "hip", "hip_runtime.h")) as f:  # the same device with 256 compute units
        text = f.read()
    assert "hipDeviceAttributeNumberOfXccs ? 8 : 1" in text
    (d / "hip" / "hip_runtime.h").write_text(text.replace("hipDeviceAttributeNumberOfXccs ? 8 : 1",
                                                          "hipDeviceAttributeNumberOfXccs ? 8 : 256"))
    (d / "driver.cpp").write_text(DRIVER)
    exe = str(d / "shapes")
    subprocess.check_call([CLANG, "-O0", "-std=c++17", "-w", "-I", str(d), "-I", csrc, str(d / "driver.cpp"),
                           os.path.join(csrc, "api.cpp"), os.path.join(csrc, "plan.cpp"), "-o", exe, "-lpthread"])

    def run(cases):
        out = subprocess.run([exe], input="".join("%d %d %d %d\n" % c for c in cases), capture_output=True, text=True)
        assert out.returncode == 0, out.stdout + out.stderr
        return out.stdout.split("\n")[:-1]
    return run


@pytest.mark.parametrize("n", [300, 512, 613])
def test_runs_of_lines(shapes, n):
    got = shapes([(n, nx, 8192 // nx, 0) for nx in (1, 2, 4, 8, 16, 64, 8192)])
    assert len(set(got)) == 1, got


def test_persistent_grid(shapes):
    """A batch of windowed lanes (tiles of 32 lines): a workgroup per tile where as many may run as the device holds,
    else no more than asked for and no more than tiles."""
    cases = [(300, 16, ny, batch) for batch in (1, 2) for ny in (2, 20, 4000)]
    assert [int(s.split()[0]) for s in shapes(cases)] == [1, 10, 2000, 1, 10, 64]
