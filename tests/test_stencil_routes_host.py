"""Which kernel a standalone stencil runs on a device of 256 compute units, by the
library's launch code on the host: the tiled kernels where their tiles are well
filled and many, the one-point-per-thread kernel for the others, which it ran
before the tiled ones and on which it is 1.05-17 times as fast there."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
DRIVER = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include "launch.h"
namespace cb {
const LineKernel *find_line_kernel(int, int, int, int, int, bool, bool) { return nullptr; }
const LineKernel *find_copy_kernel(int, int, bool) { return nullptr; }
const BatchKernel *find_batch_kernel(int, int, int, bool, bool, int, int) { return nullptr; }
const WgKernel *find_wg_kernel(int, int, int, int, bool) { return nullptr; }
const WgKernel *find_wg32_kernel(int, int, int, int, bool) { return nullptr; }
const WinKernel *find_win_kernel(int, int, int, int, bool) { return nullptr; }
const WinKernel *find_win_rows_kernel(int, int, int, int) { return nullptr; }
const WinKernel *find_win_copy_kernel(int, int, bool) { return nullptr; }
const void *stencil_kernel(int form) { return (const void *)(uintptr_t)(form + 1); }
const WinKernel *find_win_stencil_kernel(int) {
  static const WinKernel k{1, 16, 0, 2, true, 256, 2, (const void *)(uintptr_t)100, nullptr};
  return &k;
}
}  // namespace cb
hipError_t hipLaunchKernel(const void *fn, dim3, dim3, void **, size_t, hipStream_t) {
  const auto f = (uintptr_t)fn;
  puts(f == 100 ? "lanes" : (f == 1 || f == 4 ? "points" : "rows"));
  return hipSuccess;
}
int main() {
  cb_stencil st = {-2, 2, {1, 2, 0, 2, 1}};
  long n[3];
  int axis;
  while (scanf("%ld %ld %ld %d", n, n + 1, n + 2, &axis) == 4) {
    cb_grid g = {{n[0], n[1], n[2]}, {1, n[0], n[0] * n[1]}};
    const uintptr_t base = uintptr_t(1) << 40;
    if (cb_rhs_stencil(&st, &g, axis, (double *)base, (double *)(2 * base), nullptr)) return 1;
  }
}
"""
# nx, ny, nz, axis, kernel
CASES = [
    (2, 512, 4096, 1, "points"), (8, 512, 8192, 1, "points"), (24, 512, 2730, 1, "points"), (33, 512, 248, 1, "points"),
    (100, 512, 10, 1, "points"), (256, 512, 4, 1, "points"), (1000, 100, 5, 1, "points"),
    (64, 512, 1024, 1, "rows"), (128, 512, 32, 1, "rows"), (256, 256, 256, 1, "rows"), (256, 256, 256, 2, "rows"),
    (256, 200, 384, 1, "rows"), (2, 64, 512, 2, "points"), (2, 2048, 512, 2, "rows"),
    (33, 1985, 64, 0, "points"), (48, 1365, 64, 0, "points"), (65, 1008, 64, 0, "points"), (100, 328, 16, 0, "points"),
    (64, 1024, 64, 0, "lanes"), (64, 128, 64, 0, "points"), (100, 2621, 16, 0, "lanes"), (256, 256, 256, 0, "lanes"),
    (1000, 66, 16, 0, "lanes"), (1000, 33, 16, 0, "points"), (31, 5000, 64, 0, "points"),
]


def test_routes(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++ in the ROCm installation")
    csrc, host = os.path.join(ROOT, "paper_2101_02286_amd", "csrc"), os.path.join(ROOT, "tests", "host_hip")
    hip = tmp_path / "hip"
    hip.mkdir()
    with open(os.path.join(host, "hip", "hip_runtime.h")) as f:  # the same device with 256 compute units
        text = f.read()
    assert "hipDeviceAttributeNumberOfXccs ? 8 : 1" in text
    (hip / "hip_runtime.h").write_text(text.replace("hipDeviceAttributeNumberOfXccs ? 8 : 1",
                                                    "hipDeviceAttributeNumberOfXccs ? 8 : 256"))
    (tmp_path / "driver.cpp").write_text(DRIVER)
    exe = str(tmp_path / "routes")
    subprocess.check_call([CLANG, "-O0", "-std=c++17", "-w", "-I", str(tmp_path), "-I", csrc, str(tmp_path / "driver.cpp"),
                           os.path.join(csrc, "api.cpp"), os.path.join(csrc, "plan.cpp"), "-o", exe, "-lpthread"])
    out = subprocess.run([exe], input="".join("%d %d %d %d\n" % c[:4] for c in CASES), capture_output=True, text=True)
    got = out.stdout.split("\n")[:-1]
    assert out.returncode == 0 and len(got) == len(CASES)
    assert [c[:4] + (g,) for c, g in zip(CASES, got)] == CASES
