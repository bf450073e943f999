"""Where calls of automatic FP64 plans run on a device of 256 compute units: the rule
of csrc/route.h at measured points, windowed lanes (W) or the general kernel (G),
whichever was faster there."""
import os
import re
import subprocess

import pytest

from paper_2101_02286_amd import cb, schemes, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = r"""
#include <cstdio>
#include "route.h"
int main(int argc, char **) {
  int r, n, s, st, rows, cyc, uni, gM, gL, M, L, extra, run;
  long lines, blocks;
  while (scanf("%d %d %d %d %d %d %d %d %d %d %d %d %ld %ld %d", &r, &n, &s, &st, &rows, &cyc, &uni, &gM, &gL, &M, &L, &extra,
               &lines, &blocks, &run) == 15)
    puts(cb::general_is_faster({r, n, !!s, !!st, !!rows, !!cyc, !!uni, gM, gL, M, L, extra, lines, blocks, !!run, 256, argc < 2}) ? "G" : "W");
}
"""
# kernel, scheme, n, axis, log2 of the points, derivative or solve, lines: cyclic, acyclic, per-row
MEASURED = """
G tri6 56 x 25 solve cyclic        G tri6 112 x 22 solve cyclic      W tri6 144 x 22 solve cyclic
W tri6 80 x 25 solve cyclic        G tri6 124 x 22 solve cyclic      W tri6 300 x 22 solve cyclic
W tri6 613 x 16 deriv cyclic       G penta10 116 x 22 solve cyclic   W penta10 132 x 22 solve cyclic
W penta10 300 x 25 deriv cyclic    G penta10 196 x 19 solve cyclic   W penta10 196 x 25 solve cyclic
G hept12 120 x 22 deriv cyclic     W hept12 152 x 22 deriv cyclic    G hept12 152 x 22 solve cyclic
W tri6 512 y 22 deriv cyclic       W tri6 300 y 15 solve cyclic      G tri6 96 y 19 deriv cyclic
W tri6 96 y 24 deriv cyclic        W tri6 96 y 20 solve cyclic       G penta10 96 y 20 deriv cyclic
W penta10 96 y 24 deriv cyclic     W penta10 256 y 17 deriv cyclic   G penta10 200 y 17 solve cyclic
W penta10 200 y 22 solve cyclic    G penta10 1000 y 19 deriv cyclic  W penta10 1000 y 22 deriv cyclic
G hept12 128 y 22 deriv cyclic     W hept12 128 y 25 solve cyclic    G hept12 250 y 25 solve cyclic
G hept12 900 y 20 solve cyclic     W hept12 900 y 22 solve cyclic    W hept12 384 y 17 solve cyclic
W tri6 300 y 17 solve acyclic      G penta10 256 y 22 solve acyclic  W penta10 613 y 22 solve acyclic
G tri6 300 x 17 solve per-row      W tri6 300 x 22 solve per-row     G penta10 300 x 17 solve per-row
W penta10 300 x 22 solve per-row   G hept12 512 x 19 solve per-row   W hept12 512 x 22 solve per-row
W penta10 300 y 17 solve per-row   G penta10 80 y 20 solve per-row   W penta10 80 y 22 solve per-row
"""
# the same on planes of 89 lines, whose rows share 64-byte halves of cache lines
ODD = """
W tri6 192 y 22 deriv cyclic       G tri6 384 y 19 deriv cyclic      W penta10 96 y 22 deriv cyclic
G penta10 96 y 20 deriv cyclic     W penta10 384 y 23 deriv cyclic   W penta10 127 y 23 deriv cyclic
W penta10 60 y 23 deriv cyclic     G penta10 500 y 19 deriv cyclic   W penta10 1000 y 21 deriv cyclic
W hept12 64 y 23 solve cyclic      G hept12 128 y 20 deriv cyclic    W hept12 128 y 23 deriv cyclic
W hept12 500 y 22 deriv cyclic     W hept12 512 y 23 solve cyclic    W hept12 80 y 19 deriv cyclic
W penta10 127 y 23 solve acyclic   W penta10 128 y 23 solve acyclic  W hept12 153 y 22 solve acyclic
"""


def waves(r, m, lanes, d):
    """Wavefronts of a unit-stride workgroup with coefficients in LDS (win_rows_waves in csrc/plan.h)."""
    table = lanes * ((((m - r) * (4 * r + 1) + r * r) | 1) + (2 * d + 1) * r * r)
    wave = 64 // lanes * (4 * r * (lanes + 2 * d + 2) + 2 * ((lanes * (m + 1) + 4) & ~1))
    on = [(min(8, v * (163840 // (8 * (table + v * wave)))), v) for v in (4, 8, 7, 6, 5, 3, 2, 1)]
    return max(on, key=lambda t: t[0])[1]


def case(scheme, n, axis, log2, kind, lines, halves=True):
    bands = schemes.bands(scheme)
    r = (len(bands) - 1) // 2
    rows = lines == "per-row"
    plan = cb.Plan(synth.random_bands(n, r, seed=1) if rows else bands, n, cyclic=lines == "cyclic", per_row=rows,
                   host_only=True)
    strided = axis != "x"
    m, lanes, _, extra, d, _ = [int(v) for v in plan.array(13, int(strided))]
    info, s = plan.info(), "_strided" if strided else ""
    seg = plan.array(11, 0)
    if strided:
        try:
            seg = plan.array(11, 1)
        except cb.CbError:
            pass
    plan.close()
    count = 2 ** log2 // n
    if strided:
        pairs = 32 if lanes * 32 <= ((1024 if r == 3 else 512) if rows else 256) else 16
        if not halves:
            pairs = 16 if lanes * 32 > 1024 or (m == 8 and lanes > 12) else 32
        blocks = -(-(count // 2) // pairs)
    elif rows:
        blocks = -(-count // (2 * waves(r, m, lanes, d) * (64 // lanes)))
        if r == 3 or lanes >= 32:
            blocks = -(-blocks // min(3, max(1, blocks // 1024)))
    else:
        width = lanes if lanes * m == n else lanes + 2 * (d + 1)
        blocks = -(-count // ((4 if r == 1 else 1) * (64 // width)))
    return [r, n, int(strided), int(kind == "deriv"), int(rows), int(lines == "cyclic"), int(seg[7]),
            info["rows_per_lane" + s], info["lanes" + s], m, lanes, extra, count, blocks, 0]


def routes(tmp_path, table, halves):
    """The table's points, and the same with the letters that the rule gives."""
    points = [p.split() for ln in table.strip().split("\n") for p in re.split(r" {2,}", ln.strip())]
    args = [case(s, int(n), ax, int(t), kind, lines, halves) for _, s, n, ax, t, kind, lines in points]
    (tmp_path / "routes.cpp").write_text(DRIVER)
    exe = str(tmp_path / "routes")
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2101_02286_amd", "csrc"),
                           str(tmp_path / "routes.cpp"), "-o", exe])
    out = subprocess.run([exe] + ([] if halves else ["odd"]), input="\n".join(" ".join(map(str, a)) for a in args),
                         capture_output=True, text=True)
    got = out.stdout.split()
    assert len(got) == len(points)
    return [" ".join(p) for p in points], [" ".join([g] + p[1:]) for g, p in zip(got, points)]


def test_measured_points(tmp_path):
    want, got = routes(tmp_path, MEASURED, True)
    assert len(want) == 45
    assert got == want


def test_rows_that_share_half_lines(tmp_path):
    want, got = routes(tmp_path, ODD, False)
    assert got == want


@pytest.mark.parametrize("n", [129, 200, 250, 256])
def test_short_per_row_lines(n):
    """Tridiagonal unit-stride lines of up to 256 rows that 12 does not divide, heptadiagonal ones of less than
    128: the general kernels, without tables."""
    for r, m in ((1, n), (3, n // 2)):
        plan = cb.Plan(synth.random_bands(m, r, seed=1), m, per_row=True, host_only=True)
        assert len(plan.array(13, 0)) == 0 or m == 128
        plan.close()
