// Where the general kernels (line.h) are faster than windowed lanes (win.h): the
// calls of automatic FP64 one-partition plans that keep them.  Every line here
// lies between measured points of both sides (fields of 2^15-2^25 points, about
// 80 line lengths, sixth-, tenth- and twelfth-order bands, solves and fused
// derivatives); figures are time on the general kernel : time on windowed lanes.
#pragma once
#include <cstdint>

namespace cb {

struct RouteCase {
  int r, n;
  bool strided, stencil, rows, cyclic;  // rows: lanes with coefficients of their own
  bool uniform;                         // the general layout: lanes alike, their rows and count
  int gM, gL;
  int M, L, extra;                      // the windowed lanes (WinLayout)
  int64_t lines, blocks;                // of the call; workgroups of its windowed launch
  bool run;                             // the lines are one contiguous run
  int cus;                              // compute units of the device
  bool halves = true;                   // rows begin and end on 64-byte halves of cache lines
};

// Lanes with coefficients of their own: a workgroup copies its lines' tables to
// LDS first (10-90 KB), which a launch of few workgroups waits for (unit-stride
// n = 300, r = 2: 5.5 : 8.6 us at 2^17 points, 21 : 10 at 2^22).
inline bool general_rows(const RouteCase &c) {
  const int64_t cu = c.cus, b = c.blocks;
  if (!c.strided) {
    if (c.r == 1) return c.n <= 256 ? b < cu : 4 * b < 3 * cu;         // n = 300 0.88 at 109 workgroups, 1.17 at 219
    if (c.n <= 128) return b < cu + cu / 2;                  // n = 128, r = 2 0.80 at 256, 1.26 at 1024
    if (c.n == c.gM * c.gL) return 2 * b <= cu;              // n = 512, r = 3 0.61 at 64, 0.96 at 128, 1.60 at 256
    return (c.r == 2 && c.n <= 256 ? 2 : 3) * b < cu;        // r = 2, n = 250 0.86 at 100, 1.13 at 400; n = 800 0.79 at 66
  }
  // strided: long lanes, or lanes of two sizes, against general lines of few lanes
  if (c.gL == 8 && c.r == 3) return b < (c.n > 100 ? 4 : 1) * cu;           // n = 124: 0.74 at 530; n = 80: 0.71-0.81
  if (c.gL == 8) return b < cu && (c.M == 16 || (c.r == 2 && c.extra > 0));  // n = 80, r = 2: 0.77-0.89
  if (c.gL == 16) return c.r == 3 ? c.n > 192 && 4 * b < cu : c.M == 16 && 2 * b < cu;   // n = 200, r = 1: 0.78-0.90
  return c.gL == 64 && c.r == 2 && c.L >= 50 && !c.run && 4 * b < cu;                    // n = 1000: 0.91-0.94
}

inline bool general_unit_stride(const RouteCase &c) {
  const int64_t cu = c.cus, points = c.lines * c.n;
  const bool odd = c.n % 2 != 0;  // odd lengths cost the general kernel its aligned accesses
  if (c.L * c.M == c.n) {
    // many short lines in a wavefront, their tiles full of bank conflicts: n = 56 (7 lanes
    // of 8 rows) 0.75, n = 112 (7 of 16) 0.68, n = 60 (5 of 12) 0.69; 12 of 12 1.26
    const bool many = c.lines > (c.stencil && (c.L >= 6 || c.r > 1) ? 512 : 64) * cu;
    if (c.r == 1) {
      if (c.M >= 20) return c.blocks < cu;  // n = 1000: 0.93 at 128 workgroups, 1.15 at 8192
      if (c.M == 16) return c.L < 16;       // n = 176 0.89, n = 224 0.96, n = 448 1.12
      if (c.M == 12) return many && c.L < 11;
      if (c.M == 10) return many && (c.L < 8 || c.L == 9 || c.L == 11);  // n = 90 0.85, n = 100 0.99-1.12
      return many && c.L < 16;
    }
    if (c.L < 4 && many) return true;  // n = 36, r = 2: 0.76
    if (c.r == 2 && c.M >= 12 && c.L < 6 && c.lines > 256 * cu) return true;  // n = 60 0.88
    return !c.stencil && c.gM == 8 && c.M >= 12 && c.n < 420 && c.blocks < cu + cu / 2;  // n = 176, r = 2: 0.86 at 298, 1.06 at 596
  }
  // rings: halo lanes beside few lanes of the line's own
  if (c.r == 1) return c.M >= 12 && !odd && c.n < 256 && (c.n < 128 || points < (c.stencil ? 2048 : 65536) * cu);  // n = 124 0.88-1.01, 188 0.90-1.05
  if (c.r == 2) {  // n = 102-126 0.72-0.91; 24-row lanes of n = 196 0.91 at 2^19 points, 1.16 at 2^25
    if (c.n < 128 || (c.M >= 20 && c.L < 16 && c.blocks < (c.M == 20 && !odd ? 32 : 4) * cu)) return true;
    return c.M >= 16 && c.L < 32 && 2 * c.blocks < (c.stencil ? 1 : 3) * cu;
  }
  if (c.L < 9) return !c.stencil || points >= 4000 * cu;  // n = 120 0.85-0.93, derivatives 0.82-0.95
  return !c.stencil && c.n <= 192 && !odd && points >= 8192 * cu;  // n = 152 0.90, derivatives up to 1.55
}

inline bool general_strided(const RouteCase &c) {
  const int64_t cu = c.cus, points = c.lines * c.n;
  const bool few = 9 * c.blocks < 4 * cu;      // latency of a tile shows
  const bool mixed = c.extra > 0 || !c.cyclic;  // lanes read window rows of their own
  const bool full = c.n > 0.94 * c.gL * c.gM;   // little of the general layout idle
  // rows whose segments share 64-byte halves with their neighbours' (planes of 52 or 89
  // lines): windowed lanes are faster from 2^22 points on whatever the lines (n = 96,
  // r = 2 derivatives 1.37, n = 512, r = 3 solves 1.2-1.8, n = 127, r = 2 acyclic 1.4-2.2)
  if (!c.halves) {
    if (points >= 12000 * cu) return false;
    // a tile of long lanes for every ninth compute unit or fewer: n = 500 0.63-0.65 at
    // 17 tiles, n = 384-448 0.67-0.72 at 21 (whole halves of lines 0.97-1.2)
    if (c.r < 3 && c.gL == 32 && c.gM < 32 && c.L >= 24 && 9 * c.blocks < cu) return true;
    // n = 1000: 0.70-0.79 at 17 tiles, 1.17-1.26 at 65
    if (c.r == 2 && c.gL == 64) return !c.run && 6 * c.blocks < cu;
    if (c.r == 3 && c.gL == 8 && few && c.n <= 112) return false;  // n = 80: 1.19-1.21 at 103
  }
  if (c.stencil && c.M == 8 && c.extra > 0 && c.n > 56 && c.n < 64) return c.r < 3 && points >= 8000 * cu;  // 0.82-0.95
  // uniform general lanes of 12 rows, derivatives: n = 96, r = 1 0.89-0.93 up to 2^21 points,
  // 1.11 at 2^24; r = 2 0.71-0.91 up to 2^22, 1.06 at 2^24
  const bool twelve = c.uniform && c.gM == 12 && c.n >= 48;
  if (c.r == 1) return twelve && c.stencil && points < (c.n <= 384 ? 16384 : 12000) * cu;
  if (c.r == 2) {
    if (twelve && c.stencil) return points < (c.n <= 384 ? 32768 : 12000) * cu;
    if (twelve) return c.n <= 192 && points < (c.n < 64 ? 20000 : 8192) * cu;       // solves, n = 48 0.87-1.0, 96 0.81-0.90
    if (!c.cyclic && c.gL <= 8 && c.n > 52 && c.blocks < cu + cu / 2) return true;  // n = 112 0.86-0.89 up to 290
    if (!c.cyclic && c.gL <= 8 && full && c.n >= 64) return points < 20000 * cu;    // n = 64 0.81 at 2^22 points, n = 128 on 56-line planes 1.4 at 2^23
    if (c.extra > 0 && full && c.gL <= 8 && c.n > 64) return c.stencil || points < 8192 * cu;  // n = 124 0.82-0.97
    if (!c.cyclic && c.n == c.gL * c.gM && c.gL == 16) return points < 20000 * cu;  // n = 256 0.87-0.92, 1.2 at 2^24
    // n = 92 0.88, 200 0.88-0.93 at 2^17 points; n = 1000 0.80 up to 2^20, 1.57 at 2^22
    if (mixed && few && c.gL >= 8 && c.gL < 32) return true;
    if (mixed && c.gL == 64 && !c.run && 3 * c.blocks < cu) return true;
    return c.stencil && c.gL == 64 && c.L >= 48 && !c.run && 4 * c.blocks < cu;     // n = 800 0.92
  }
  if (c.uniform) {  // n = 128 derivatives 0.63-0.94; solves 0.74-0.88 up to 2^22 points, 1.04 at 2^25
    if (c.n > 512) return points < (c.stencil ? 32768 : 16384) * cu;
    if (c.n <= 32) return c.stencil && points < 16384 * cu;
    return c.stencil || points < 65536 * cu;
  }
  if (mixed && c.gL <= 16) {
    if (full) return true;                                // n = 127 0.70-0.90, n = 250 0.77-0.90
    if (!c.cyclic && c.gL == 8) return points < (c.n > 108 ? 131072 : 32768) * cu;  // n = 112 0.80-0.91, n = 80 0.89 at 2^22
    if (c.extra > 0 && c.L < 12 && points < 65536 * cu && c.n > 144) return true;   // n = 153 0.80-0.94, 2^25 1.16
    return c.blocks < cu + cu / 2;                        // n = 200 0.77-0.90 at up to 326 workgroups, 1.17 at 650
  }
  if (c.stencil && c.extra > 0 && c.gL == 32 && full) return true;  // n = 500 0.83-0.97 (rows of 96 lines 1.1-1.3)
  if (!c.cyclic && c.gL == 32 && full) return c.blocks < cu;  // n = 512 0.87-0.93 up to 128
  if (c.gL == 64) return !c.run && (mixed ? 3 * c.blocks < cu : c.L >= 50 && c.L < 60 && 4 * c.blocks < cu);  // n = 1000
  return few && (c.gL < 32 || mixed);                         // 0.67-0.70 up to 2^21 points, 1.35 at 2^22
}

inline bool general_is_faster(const RouteCase &c) {
  return c.rows ? general_rows(c) : (c.strided ? general_strided(c) : general_unit_stride(c));
}

}  // namespace cb
