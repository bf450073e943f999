// Windowed-lane kernels: constant-band lines of any length whose inverse
// decays (WinLayout in plan.h).  Included by the win_*.hip instance files.
//
// k_line's general layouts (line lengths that are no power of two times a
// kernel's row count) were bound by latency: every lane read its coefficients
// from LDS, log2 L exchanges ran one after the other, each behind a barrier,
// and 112-127 VGPRs left four wavefronts per SIMD.  Here every row's
// coefficients come through the scalar cache for lanes of any size, one
// exchange solves the reduced system, and a lane's rows never leave their
// registers, so what is left is memory: whole rows of 128-byte lines run at
// 300-390 GDOF/s (4.8-6.2 TB/s), rows that share lines with their neighbours
// at 230-310, where the requests to L2 are the limit (a 256-byte segment at an
// odd offset takes three lines instead of two).  GDOF/s of the FP64 fused
// derivative before -> after, x / y / z:
//   500 x 613 x 338    sixth order  302 / 159 / 171 -> 371 / 306 / 297
//   543 x 215 x 958    tenth order  104 / 149 / 121 -> 310 / 272 / 250
// and of the solve of 2500 x 115 x 115 lines along x, sixth order 199 -> 345,
// tenth order 94 -> 326 (chunks of lanes that recompute D + 1 lanes of their
// neighbours instead of three launches that pass them through memory).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"
#include "launch.h"

namespace cb {

// Strided rows are read and written as pairs of adjacent lines, one pair per
// thread: 16 bytes per access, coefficients fetched once for both lines, two
// chains of dependent operations in flight (16 rows of two lines instead of 32
// of one, 512^3 sixth order y / z 341 / 324 -> 355 / 348 GDOF/s).  Unit-stride
// rows one line per thread.
typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));  // any 8-byte address
template <int NL> struct WinVec { typedef double type; };
template <> struct WinVec<2> { typedef dbl2 type; };

constexpr int win_lines(int mode) { return mode == MODE_S ? 2 : 1; }  // lines per thread

// LDS planes, one value per thread and plane: the halo of Q rows per side that
// strided rows exchange for the stencil, and what a lane shares for the reduced
// system (2R).  Where both together would leave one workgroup to a compute unit,
// the second takes the first's place behind a barrier of its own.
constexpr int win_halo_planes(int Q, int mode) { return mode == MODE_S ? 2 * Q : 0; }
constexpr bool win_shared_planes(int R, int Q, int mode) {
  return mode == MODE_S && win_halo_planes(Q, mode) + 2 * R >= 8;
}
constexpr int win_planes(int R, int Q, int mode) {
  const int h = win_halo_planes(Q, mode);
  return win_shared_planes(R, Q, mode) ? (h > 2 * R ? h : 2 * R) : h + 2 * R;
}

// Position of a thread: lane l of the Lw its line (or pair of lines) has in the
// workgroup.  A plane holds, per line, the lanes' values between D + 1 spare
// ones on either side: of a line that is whole the far lanes' again, so that
// neighbours lie at a fixed distance (step) without a wrap; of a chunk nothing
// that a stored lane depends on.
struct WinPos {
  int l, Lw, D, at, step, NS;  // at: the lane's slot; NS: slots per plane
  bool live, whole, block;
  __device__ __forceinline__ void sync() const {
    if (block) {
      __syncthreads();
    } else {  // a line's lanes lie in one wavefront, whose LDS traffic is in order
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
  // share CNT values with the lanes up to `reach` away
  template <int CNT, typename V>
  __device__ __forceinline__ void publish(V *ex, const V (&v)[CNT], int reach) const {
    if (live) {
#pragma unroll
      for (int i = 0; i < CNT; ++i) ex[i * NS + at] = v[i];
      if (whole && l < reach) {
#pragma unroll
        for (int i = 0; i < CNT; ++i) ex[i * NS + at + Lw * step] = v[i];
      }
      if (whole && l >= Lw - reach) {
#pragma unroll
        for (int i = 0; i < CNT; ++i) ex[i * NS + at - Lw * step] = v[i];
      }
    }
    sync();
  }
};

// x~_l = sum_{|d| <= D} g[d] (c_{l+d} - t_{l+d-1}), the lane's window of the
// reduced system's inverse, and x~_{l+1} by the same window one lane on (a
// second exchange would cost a barrier).  ct: c and t of Eq. (21).  g: one row
// for the whole wavefront, read through the scalar cache ahead of the barrier.
template <int R, int D, typename V>
__device__ __forceinline__ void win_reduce(const double *g, const WinPos &p, V *ex, const V (&ct)[2 * R], V (&xt)[R],
                                           V (&xn)[R]) {
  double gm[(2 * D + 1) * R * R];
#pragma unroll
  for (int i = 0; i < (2 * D + 1) * R * R; ++i) gm[i] = cld(g + i);
  p.publish(ex, ct, D + 1);
#pragma unroll
  for (int a = 0; a < R; ++a) xt[a] = xn[a] = (V)0.0;
#pragma unroll
  for (int d = -D; d <= D + 1; ++d) {
#pragma unroll
    for (int b = 0; b < R; ++b) {
      const V v = ex[b * p.NS + p.at + d * p.step] - ex[(R + b) * p.NS + p.at + (d - 1) * p.step];
#pragma unroll
      for (int a = 0; a < R; ++a) {
        if (d <= D) xt[a] += gm[(d <= D ? d + D : 0) * R * R + a * R + b] * v;
        if (d > -D) xn[a] += gm[(d > -D ? d - 1 + D : 0) * R * R + a * R + b] * v;
      }
    }
    // (a few reads in flight at a time: the lane's rows fill the registers)
    if (R > 1 || (d + D) % 2) __builtin_amdgcn_sched_barrier(0);
  }
}
// The same for lanes that read different rows (gn: the next lane's), and for
// wide windows.  g, gn: in LDS, or uniform.
template <int R, typename V>
__device__ __forceinline__ void win_reduce_any(const double *g, const double *gn, const WinPos &p, V *ex,
                                               const V (&ct)[2 * R], V (&xt)[R], V (&xn)[R]) {
  p.publish(ex, ct, p.D + 1);
#pragma unroll
  for (int a = 0; a < R; ++a) xt[a] = xn[a] = (V)0.0;
  const int at = p.at - p.D * p.step;
  auto value = [&](int d, int b) { return ex[b * p.NS + at + d * p.step] - ex[(R + b) * p.NS + at + (d - 1) * p.step]; };
  auto add = [&](V(&x)[R], const double *row, V v, int b) {
#pragma unroll
    for (int a = 0; a < R; ++a) x[a] += row[a * R + b] * v;
  };
#pragma unroll
  for (int b = 0; b < R; ++b) add(xt, g, value(0, b), b);
#pragma unroll 1
  for (int d = 1; d <= 2 * p.D; ++d)
#pragma unroll
    for (int b = 0; b < R; ++b) {
      const V v = value(d, b);
      add(xt, g + d * R * R, v, b);
      add(xn, gn + (d - 1) * R * R, v, b);
    }
#pragma unroll
  for (int b = 0; b < R; ++b) add(xn, gn + 2 * p.D * R * R, value(2 * p.D + 1, b), b);
}

// Solve the lane's rows v (b on entry, x on exit).  sh: the lane holds M - 1
// rows.  last: the last lane of an acyclic line.  gi, gin: the lane's and the
// next lane's row of the window table g, whose copy in LDS is gl.
// ROW: the lane has coefficients of its own, at cf in LDS.
template <int R, int M, typename V, bool UNI, bool ROW>
__device__ __forceinline__ void win_solve(V (&v)[M], const double *cf, const double *g, const double *gl, int gi, int gin, const WinPos &p, V *ex,
                                          bool sh, bool last) {
  constexpr int N = M - R, RW = win_row_size(R), RR = R * R;
  const int D = p.D;
  const V zero = (V)0.0;
  auto co = [&](int i) { return ROW ? cf[i] : cld(cf + i); };
  // z = L^{-1} b on the interior rows
#pragma unroll
  for (int j = 1; j < N; ++j)
#pragma unroll
    for (int q = 1; q <= R; ++q)
      if (j - q >= 0) v[R + j] -= co(j * RW + q - 1) * v[R + j - q];
  if (!UNI) v[M - 1] = sh ? zero : v[M - 1];
  // c = b~ - U~ y_first, t = L~ y_last (Eq. (21))
  V ct[2 * R], xt[R], xn[R + 1], xr[R];
#pragma unroll
  for (int a = 0; a < R; ++a) {
    V acc = v[a];
#pragma unroll
    for (int j = 0; j < N; ++j) acc -= co(j * RW + R + a) * v[R + j];
    ct[a] = acc;
  }
  {
    V zl[R];
#pragma unroll
    for (int i = 0; i < R; ++i) zl[i] = UNI ? v[M - R + i] : (sh ? v[M - R - 1 + i] : v[M - R + i]);
#pragma unroll
    for (int a = 0; a < R; ++a) {
      V acc = zero;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const double z0 = co(N * RW + a * R + i);
        acc += (UNI || ROW ? z0 : (sh ? co(N * RW + RR + a * R + i) : z0)) * zl[i];
      }
      ct[R + a] = (!UNI && last) ? zero : acc;
    }
  }
  // x~: most wavefronts hold lanes that share one window row
  const int gu = UNI || ROW ? 0 : __builtin_amdgcn_readfirstlane(gi);
  const double *gw = g + (size_t)gu * ((2 * D + 1) * RR);
  constexpr int DF = M >= 24 ? 3 : (R == 1 ? 6 : 4);  // unrolled windows
  if (!ROW && D <= DF && (UNI || __all(gi == gu && gin == gu))) {
    if (D == 1) win_reduce<R, 1, V>(gw, p, ex, ct, xt, xr);
    else if (D == 2) win_reduce<R, 2, V>(gw, p, ex, ct, xt, xr);
    else if (D == 3) win_reduce<R, 3, V>(gw, p, ex, ct, xt, xr);
    else if (DF >= 4 && D == 4) win_reduce<R, DF >= 4 ? 4 : 1, V>(gw, p, ex, ct, xt, xr);
    else if (DF >= 5 && D == 5) win_reduce<R, DF >= 5 ? 5 : 1, V>(gw, p, ex, ct, xt, xr);
    else if (DF >= 6) win_reduce<R, DF >= 6 ? 6 : 1, V>(gw, p, ex, ct, xt, xr);
  } else {
    const double *gs = UNI ? g : gl;
    win_reduce_any<R, V>(gs + gi * ((2 * D + 1) * RR), gs + gin * ((2 * D + 1) * RR), p, ex, ct, xt, xr);
  }
#pragma unroll
  for (int a = 0; a < R; ++a) xn[a] = (!UNI && last) ? zero : xr[a];
  xn[R] = zero;
  // x = U^{-1} (z - ell x~_l), with the next lane's interface rows beyond its end
  V e[R];  // slots M .. M+R-1
#pragma unroll
  for (int a = 0; a < R; ++a) e[a] = UNI ? xn[a] : (sh ? xn[a + 1] : xn[a]);
#pragma unroll
  for (int j = N - 1; j >= 0; --j) {
    V acc = v[R + j];
#pragma unroll
    for (int a = 0; a < R; ++a) acc -= co(j * RW + 2 * R + a) * xt[a];
    acc *= co(j * RW + 3 * R);
#pragma unroll
    for (int q = 1; q <= R; ++q)
      acc -= co(j * RW + 3 * R + q) * (j + q < N ? v[j + q < N ? R + j + q : 0] : e[j + q < N ? 0 : j + q - N]);
    v[R + j] = (!UNI && j == N - 1) ? (sh ? xn[0] : acc) : acc;
  }
#pragma unroll
  for (int a = 0; a < R; ++a) v[a] = xt[a];
}

// v[k] of a lane whose rows before its first are prev[Q] and whose slots from
// M - 1 on are tail[Q + 1] (tail[0]: row M - 1, or the next lane's first row
// when the lane holds M - 1 rows).
template <int Q, int M, typename V>
__device__ __forceinline__ V win_at(const V (&v)[M], const V (&prev)[Q], const V (&tail)[Q + 1], int k) {
  if (k < 0) return prev[k + Q < 0 ? 0 : k + Q];
  if (k < M - 1) return v[k < M - 1 ? k : 0];
  return tail[k - M + 1 > Q ? Q : (k < M - 1 ? 0 : k - M + 1)];
}
template <int Q, int M, bool UNI, typename V>
__device__ __forceinline__ void win_tail(const V (&v)[M], const V (&next)[Q], bool sh, V (&tail)[Q + 1]) {
  tail[0] = UNI ? v[M - 1] : (sh ? next[0] : v[M - 1]);
#pragma unroll
  for (int i = 0; i < Q; ++i) tail[1 + i] = UNI ? next[i] : (sh ? next[i + 1 < Q ? i + 1 : i] : next[i]);
}

// Exchange of the Q rows at either end of every lane.
template <int Q, int M, bool UNI, typename V>
__device__ __forceinline__ void win_halo(const V (&v)[M], bool sh, const WinPos &p, V *ex, V (&prev)[Q], V (&next)[Q]) {
  V h[2 * Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    h[i] = v[i];
    h[Q + i] = UNI ? v[M - Q + i] : (sh ? v[M - 1 - Q + i] : v[M - Q + i]);
  }
  p.publish(ex, h, 1);
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    prev[i] = ex[(Q + i) * p.NS + p.at - p.step];
    next[i] = ex[i * p.NS + p.at + p.step];
  }
}

// A row of a pair of adjacent lines; one: only the first line exists.
template <bool NT>
__device__ __forceinline__ dbl2 win_load2(const double *q, bool one) {
  if (one) return dbl2{*q, 0.0};
  const dbl2u *s = reinterpret_cast<const dbl2u *>(q);
  return NT ? (dbl2)__builtin_nontemporal_load(s) : (dbl2)*s;
}

template <bool NT>
__device__ __forceinline__ void win_store2(dbl2 v, double *q) {
  dbl2u *s = reinterpret_cast<dbl2u *>(q);
  if (NT) __builtin_nontemporal_store((dbl2u)v, s);
  else *s = v;
}
template <bool B> struct WinFlag { static constexpr bool value = B; };

// What a tile's rows go through between their loads and their stores: the
// stencil (Q > 0) and the solve (with one set of coefficients for all lanes, or
// one for each), nothing, or the stencil alone.
enum { WIN_SOLVE = 0, WIN_MOVE = 1, WIN_STENCIL = 2, WIN_ROWS = 3 };

// One tile: the lanes of W lines (pairs of lines), or of one run of lanes
// (chunk) of each of them with H halo lanes on either side.  threads: those of
// the workgroup that run the tile (a batched launch may have more).
template <int R, int M, int MODE, int Q, bool UNI, int OP>
__device__ __forceinline__ void win_tile(const WinArgs &a, uint32_t tile, double *smem, int threads) {
  constexpr int QQ = Q > 0 ? Q : 1;
  constexpr bool ROW = OP == WIN_ROWS, SOLVE = OP == WIN_SOLVE || ROW;
  constexpr int KT = Q > 0 ? M + 2 : M;  // tile rows a lane loads (a window's halo needs one or two more)
  constexpr int NL = ROW ? 2 : win_lines(MODE);  // lines per thread
  typedef typename WinVec<NL>::type VD;
  const int tid = threadIdx.x;
  WinPos p;
  p.Lw = a.Lw;
  p.D = a.D;
  p.block = MODE == MODE_S;
  p.whole = !a.ring;
  int li;
  if (MODE == MODE_S) {
    p.l = tid >> a.lgW;
    li = tid & ((1 << a.lgW) - 1);
    p.live = p.l < a.Lw;
    p.step = 1 << a.lgW;
    p.NS = (a.Lw + 2 * a.D + 2) << a.lgW;
    p.l = p.live ? p.l : 0;
    p.at = ((p.l + a.D + 1) << a.lgW) + li;
  } else {
    const int t = tid & 63;
    const int q = (int)(((uint32_t)t * a.linv) >> 16);  // t / Lw
    p.live = q < a.lpw;
    p.l = p.live ? t - q * a.Lw : 0;
    li = (tid >> 6) * a.lpw + (p.live ? q : 0);
    p.step = 1;
    p.NS = a.W * (a.Lw + 2 * a.D + 2);
    p.at = li * (a.Lw + 2 * a.D + 2) + a.D + 1 + p.l;
  }
  const bool live = p.live;
  uint32_t ch = 0, lt = tile;
  if (a.nch > 1) {
    if (a.chunk_fast) {
      lt = tile / (uint32_t)a.nch;
      ch = tile - lt * (uint32_t)a.nch;
    } else {
      ch = tile / a.ltiles;
      lt = tile - ch * a.ltiles;
    }
  }
  constexpr int XL = MODE == MODE_X ? NL : 1;  // (strided pairs count as one line, with su = 2)
  const int64_t line = ((int64_t)lt * a.W + li) * XL;
  const bool lactive = live && line < a.nlines;
  const FastDiv fd{a.nudiv.d, a.nudiv.mul, a.nudiv.s1, a.nudiv.s2};
  const uint32_t line32 = lactive ? (uint32_t)line : 0u;
  const uint32_t lv = fd.div(line32), lu = line32 - lv * a.nudiv.d;
  const int64_t lbase = (int64_t)lu * a.su + (int64_t)lv * a.sv;
  const bool one = MODE == MODE_S && (int)lu == a.one;  // a pair with only its first line
  // the lane: g of the line's L lanes; own: lanes this tile stores, between H
  // halo lanes on either side
  const int H = a.H;
  int own = a.L - (int)ch * a.Lc;
  own = own < a.Lc ? own : a.Lc;
  int g = (int)ch * a.Lc - H + p.l;
  bool active = lactive && p.l < own + 2 * H;
  const bool store = active && p.l >= H && p.l < H + own;
  bool sh = false;
  int m = M, start = 0;
  if (MODE == MODE_S || !UNI) {
    if (a.acyclic) active = active && g >= 0 && g < a.L;
    g = g < 0 ? g + a.L : (g >= a.L ? g - a.L : g);
    g = g < 0 || g >= a.L ? 0 : g;  // (lanes past the last chunk's window)
    sh = !UNI && g >= a.extra && a.extra > 0;
    m = sh ? M - 1 : M;
    start = UNI ? g * M : g * a.base + (g < a.extra ? g : a.extra);
  }
  VD b64[M];
  VD gp[QQ], gn[QQ];
  const VD zero = (VD)0.0;
  // unit-stride lines go through an LDS tile: word e holds row r0 + e (modulo n)
  double *tb = nullptr;
  auto row = [&](int w) -> VD {
    if constexpr (XL == 2) return VD{tb[w], tb[a.pitch + w]};
    else return (VD)tb[w];
  };
  const double *lin = a.in + lbase;
  int64_t other = 0;  // unit-stride pairs: from the first line to the second
  bool two = false;
  if (XL == 2) {
    two = lactive && line + 1 < a.nlines;
    const uint32_t l1 = two ? line32 + 1 : line32, v1 = fd.div(l1), u1 = l1 - v1 * a.nudiv.d;
    other = (int64_t)u1 * a.su + (int64_t)v1 * a.sv - lbase;
  }
  int r0 = 0, len = 0;
  // (a pad word per M words: lane l's rows are words l (M + 1) + 0..M-1, free of
  // bank conflicts; halo rows before lane 0 have negative e, words -1 - |e|)
  // (lanes of two sizes: the smaller ones leave one more word unused)
  const int big = a.extra * M;
  auto at = [&](int e) {
    if (UNI) return e + (int)((uint32_t)(e + M) / (uint32_t)M) - 1;
    if (e < big || a.extra == 0) return e + (int)((uint32_t)e / (uint32_t)M);
    return a.extra * (M + 1) + (e - big) + 2 * (int)((uint32_t)(e - big) / (uint32_t)(M - 1));
  };
  constexpr int QP = (Q + 1) & ~1;  // halo rows beyond the window's lanes, kept even
  if constexpr (MODE == MODE_X) {
    tb = smem + (size_t)win_planes(R, Q, MODE) * NL * p.NS + (size_t)li * XL * a.pitch + QP + 2;
    len = a.n;
    if (a.ring) {
      r0 = ((int)ch * a.Lc - H) * M;
      len = (own + 2 * H) * M;
    }
    const int e0 = a.ring ? -QP : 0, e1 = a.ring ? len + QP : len;
    // pairs of rows from any 8-byte address (r0, len and QP are even); the ring
    // wraps between the rows of a pair when n is odd
    auto load = [&](auto nt) {
      dbl2 t2[XL][KT / 2];
#pragma unroll
      for (int h = 0; h < XL; ++h)
#pragma unroll
        for (int k = 0; k < KT / 2; ++k) {
          const int e = e0 + 2 * (p.l + k * a.Lw);
          int r = r0 + e;
          r = r < 0 ? r + a.n : (r >= a.n ? r - a.n : r);
          t2[h][k] = dbl2{0.0, 0.0};
          if ((h == 0 ? lactive : two) && e < e1) {
            const double *q = h == 0 ? lin : lin + other;
            if (r == a.n - 1) t2[h][k] = dbl2{q[r], q[0]};  // (of a whole line the second is not kept)
            else t2[h][k] = win_load2<decltype(nt)::value>(q + r, false);
          }
        }
#pragma unroll
      for (int k = 0; k < KT / 2; ++k) {
        const int e = e0 + 2 * (p.l + k * a.Lw);
        if (live && e < e1) {
          const int w = at(e), w1 = UNI ? w + 1 : at(e + 1);
#pragma unroll
          for (int h = 0; h < XL; ++h) {
            tb[h * a.pitch + w] = t2[h][k].x;
            if (UNI || e + 1 < e1) tb[h * a.pitch + w1] = t2[h][k].y;
          }
        }
      }
    };
    if (a.nt) load(WinFlag<true>());
    else load(WinFlag<false>());
    p.sync();
#pragma unroll
    for (int k = 0; k < M; ++k) b64[k] = active && (UNI || k < M - 1 || !sh) ? row(p.l * (M + 1) + k) : zero;
  } else {
    const double *in = lin + (int64_t)start * a.rs;
    if (a.nt && !one) {
#pragma unroll
      for (int k = 0; k < M; ++k)
        b64[k] = (active && (UNI || k < M - 1 || !sh)) ? win_load2<true>(in + k * a.rs, false) : zero;
    } else if (!one) {
#pragma unroll
      for (int k = 0; k < M; ++k)
        b64[k] = (active && (UNI || k < M - 1 || !sh)) ? win_load2<false>(in + k * a.rs, false) : zero;
    } else {
#pragma unroll
      for (int k = 0; k < M; ++k)
        b64[k] = (active && (UNI || k < M - 1 || !sh)) ? win_load2<false>(in + k * a.rs, true) : zero;
    }
    if (Q > 0 && SOLVE) {
      // the window's ends take their halo from memory
#pragma unroll
      for (int i = 0; i < QQ; ++i) {
        gp[i] = gn[i] = zero;
        if (a.ring && active && p.l == 0) {
          const int r = start - Q + i;
          gp[i] = win_load2<false>(lin + (int64_t)(r < 0 ? r + a.n : r) * a.rs, one);
        }
        if (a.ring && active && p.l == own + 2 * H - 1) {
          const int r = start + m + i;
          gn[i] = win_load2<false>(lin + (int64_t)(r >= a.n ? r - a.n : r) * a.rs, one);
        }
      }
    }
  }
  // lanes of two sizes read different rows of the window table: copied to LDS
  // (visible after the next exchange)
  double *gl = smem + (size_t)win_planes(R, Q, MODE) * NL * p.NS + (MODE == MODE_X ? (size_t)a.W * XL * a.pitch : 0);
  if (!UNI && OP == WIN_SOLVE) {
    const double *gw = static_cast<const double *>(a.g);
    for (int i = tid; i < a.gcount; i += threads) gl[i] = gw[i];
  }
  if (Q > 0 && OP != WIN_MOVE) {  // fused right-hand-side stencil (Eqs. (1)-(2)), periodic
    VD fp[QQ], fn[QQ], tail[QQ + 1];
    if constexpr (MODE == MODE_X) {
#pragma unroll
      for (int i = 0; i < QQ; ++i) {
        // the last rows of the lane before and the first of the next one
        int e = p.l * (M + 1) - 1 - Q + i, f = (p.l + 1) * (M + 1) + i;
        if (p.l == 0 && !a.ring) e = a.Lw * (M + 1) - 1 - Q + i;
        if (p.l == a.Lw - 1 && !a.ring) f = i;
        if (!UNI && a.extra > 0 && (p.l == 0 || p.l > a.extra)) --e;  // the lane before holds M - 1 rows
        fp[i] = active ? row(e) : zero;
        fn[i] = active ? row(f) : zero;
      }
    } else {
      win_halo<QQ, M, UNI, VD>(b64, sh, p, reinterpret_cast<VD *>(smem), fp, fn);
      if (a.ring) {
#pragma unroll
        for (int i = 0; i < QQ; ++i) {
          fp[i] = p.l == 0 ? gp[i] : fp[i];
          fn[i] = p.l == own + 2 * H - 1 ? gn[i] : fn[i];
        }
      }
    }
    win_tail<QQ, M, UNI, VD>(b64, fn, sh, tail);
    VD bb[M];
#pragma unroll
    for (int k = 0; k < M; ++k) {
      VD acc = zero;
#pragma unroll
      for (int q = -Q; q <= Q; ++q)  // (the stencil by itself: its own taps only, as 0 x inf is not 0)
        if (SOLVE || (q >= a.lo && q <= a.hi)) acc += a.stc[q + 3] * win_at<QQ, M, VD>(b64, fp, tail, k + q);
      bb[k] = (!UNI && k == M - 1 && sh) ? zero : acc;
    }
#pragma unroll
    for (int k = 0; k < M; ++k) b64[k] = bb[k];
  }
  if (SOLVE) {
    const double *cf = static_cast<const double *>(a.coef);
    const double *gw = static_cast<const double *>(a.g);
    const int gi = UNI ? 0 : a.gidx[g], gin = UNI ? 0 : a.gidx[g + 1 < a.L ? g + 1 : 0];
    const bool last = !UNI && a.acyclic && g == a.L - 1;
    constexpr bool shared = win_shared_planes(R, Q, MODE);
    constexpr int HP = win_halo_planes(Q, MODE) * NL;
    VD *ex = reinterpret_cast<VD *>(smem + (shared ? 0 : (size_t)HP * p.NS));
    if (shared && Q > 0) p.sync();  // the halo has been read
    if (ROW) {  // (stride odd: no bank conflicts between a line's lanes)
      win_solve<R, M, VD, UNI, true>(b64, gl + a.gcount + (p.live ? g : 0) * win_lane_size(R, M), gw, gl, gi, gin, p, ex, sh, last);
    } else {
      win_solve<R, M, VD, UNI, false>(b64, cf, gw, gl, gi, gin, p, ex, sh, last);
    }
  }
  if constexpr (MODE == MODE_X) {
    if (!SOLVE) p.sync();  // (the solve's exchange lies in between)
#pragma unroll
    for (int k = 0; k < M; ++k)
      if (active && (UNI || k < M - 1 || !sh)) {
        if constexpr (XL == 2) {
          tb[p.l * (M + 1) + k] = b64[k].x;
          tb[a.pitch + p.l * (M + 1) + k] = b64[k].y;
        } else {
          tb[p.l * (M + 1) + k] = b64[k];
        }
      }
    p.sync();
    double *lout = a.out + lbase;
    int s0 = 0, s1 = len;  // tile words this tile stores
    if (a.ring) {
      s0 = H * M;
      const int rows = a.n - (int)ch * a.Lc * M;
      s1 = s0 + (rows < own * M ? rows : own * M);
    }
    auto put = [&](auto nt) {
#pragma unroll
      for (int k = 0; k < KT / 2; ++k) {
        const int e = 2 * (p.l + k * a.Lw);
        if (lactive && e >= s0 && e < s1) {
          const int w = at(e), w1 = UNI ? w + 1 : at(e + 1);
#pragma unroll
          for (int h = 0; h < XL; ++h) {
            if (h == 1 && !two) continue;
            double *q = lout + (h == 0 ? 0 : other) + r0 + e;
            const double *t = tb + h * a.pitch;
            if (e + 1 == s1) *q = t[w];
            else win_store2<decltype(nt)::value>(dbl2{t[w], t[w1]}, q);
          }
        }
      }
    };
    if (a.nt) put(WinFlag<true>());
    else put(WinFlag<false>());
  } else {
    if (!store) return;  // (no barrier follows in the tile)
    // (the output row as a distance from the input row: one address stays live)
    double *out = const_cast<double *>(lin) + (a.out - a.in) + (int64_t)start * a.rs;
    if (a.nt && !one) {
#pragma unroll
      for (int k = 0; k < M; ++k)
        if (UNI || k < M - 1 || !sh) win_store2<true>(b64[k], out + k * a.rs);
    } else if (!one) {
#pragma unroll
      for (int k = 0; k < M; ++k)
        if (UNI || k < M - 1 || !sh) win_store2<false>(b64[k], out + k * a.rs);
    } else {
#pragma unroll
      for (int k = 0; k < M; ++k)
        if (UNI || k < M - 1 || !sh) out[k * a.rs] = b64[k].x;
    }
  }
}

// Workgroup bound of an instance: unit-stride ones run 256 threads.
template <int MODE>
constexpr int win_max_threads() {
  return MODE == MODE_X ? 256 : 1024;
}

template <int MODE>
constexpr int win_rows_threads() {
  return MODE == MODE_X ? 512 : 1024;
}

template <int R, int M, int MODE, int Q, bool UNI, int OP = WIN_SOLVE>
__global__ __launch_bounds__((win_max_threads<MODE>()), 4) void k_win(const WinArgs a) {
  extern __shared__ __align__(16) double smem[];
  uint32_t tile = blockIdx.x;
  if (a.xcds > 1) {  // tiles grouped by XCD, as in k_line
    const uint32_t X = (uint32_t)a.xcds, G = gridDim.x, q = G / X, rem = G % X;
    const uint32_t j = tile % X, s = tile / X;
    tile = j * q + (j < rem ? j : rem) + s;
  }
  win_tile<R, M, MODE, Q, UNI, OP>(a, tile, smem, (int)blockDim.x);
}

// Lanes with coefficients of their own: bands that vary by row.  The lanes'
// coefficients and windows lie in LDS, copied once for a.run tiles, and every
// thread takes two lines, unit-stride ones too: these are bound by LDS reads
// (4R + 1 words a row, one line per thread 156 GDOF/s at r = 2, n = 300, two
// 196), which the memory path of strided lines hides (301).  Unit-stride
// workgroups fill a compute unit's LDS with two wavefronts per SIMD, so the
// registers of four are theirs.
template <int R, int M, int MODE, int Q>
__global__ __launch_bounds__((win_rows_threads<MODE>()), (MODE == MODE_X ? 2 : 4)) void k_win_rows(const WinArgs a) {
  extern __shared__ __align__(16) double smem[];
  uint32_t blk = blockIdx.x;
  if (a.xcds > 1) {  // grouped by XCD, as in k_line
    const uint32_t X = (uint32_t)a.xcds, G = gridDim.x, q = G / X, rem = G % X;
    const uint32_t j = blk % X, s = blk / X;
    blk = j * q + (j < rem ? j : rem) + s;
  }
  const int NS = a.W * (a.Lw + 2 * a.D + 2);
  double *gl = smem + (size_t)win_planes(R, Q, MODE) * 2 * NS + (MODE == MODE_X ? (size_t)a.W * 2 * a.pitch : 0);
  for (int i = threadIdx.x; i < a.gcount; i += blockDim.x) gl[i] = a.g[i];
  const int words = a.L * win_lane_size(R, M);
  for (int i = threadIdx.x; i < words; i += blockDim.x) gl[a.gcount + i] = a.coef[i];
  __syncthreads();
  for (int i = 0; i < a.run; ++i) {
    const uint32_t tile = blk * (uint32_t)a.run + (uint32_t)i;
    if (tile >= a.ltiles) break;
    if (i > 0) __syncthreads();  // (the tile before has read the planes)
    win_tile<R, M, MODE, Q, false, WIN_ROWS>(a, tile, smem, (int)blockDim.x);
  }
}

// Batched launch over the tiles of many items of one instance, as k_batched.
// Wavefronts beyond an item's own workgroup size leave at once (a barrier
// counts the wavefronts that remain) or, in the persistent form, idle.
template <int R, int M, int MODE, int Q, bool UNI>
__global__ __launch_bounds__((win_max_threads<MODE>()), 4) void k_win_batched(BatchHdr *hdr,
                                                                             const WinItemDev *__restrict__ items,
                                                                             int per_tile) {
  extern __shared__ __align__(16) double smem[];
  const int64_t total = hdr->total_tiles;
  const int nitems = hdr->n_items;
  auto item_of = [&](int64_t t) {
    int lo = 0, hi = nitems - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (items[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  if (per_tile) {
    const int64_t t = blockIdx.x;
    if (t >= total) return;
    const int i = item_of(t);
    const WinItemDev &it = items[i];
    if ((int)threadIdx.x >= it.threads) return;
    uint32_t local = (uint32_t)(t - it.tile_begin);
    if (it.a.xcds > 1) {
      const uint32_t G = (uint32_t)((i + 1 < nitems ? items[i + 1].tile_begin : total) - it.tile_begin);
      const uint32_t X = (uint32_t)it.a.xcds, q = G / X, rem = G % X, j = local % X, s = local / X;
      local = j * q + (j < rem ? j : rem) + s;
    }
    win_tile<R, M, MODE, Q, UNI, WIN_SOLVE>(it.a, local, smem, it.threads);
    return;
  }
  for (;;) {
    unsigned long long *next = reinterpret_cast<unsigned long long *>(smem);
    if (threadIdx.x == 0) *next = atomicAdd(&hdr->next_tile, 1ull);
    __syncthreads();
    const int64_t t = (int64_t)*next;
    __syncthreads();
    if (t >= total) break;
    const WinItemDev &it = items[item_of(t)];
    win_tile<R, M, MODE, Q, UNI, WIN_SOLVE>(it.a, (uint32_t)(t - it.tile_begin), smem, (int)blockDim.x);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    __threadfence();
    const unsigned prev = atomicAdd(&hdr->done, 1u);
    if (prev == gridDim.x - 1) {
      atomicExch(&hdr->next_tile, 0ull);
      atomicExch(&hdr->done, 0u);
      __threadfence();
    }
  }
}

template <int R, int M, int MODE, int Q, bool UNI>
const void *win_batched() {
  if constexpr (Q > 0) return (const void *)&k_win_batched<R, M, MODE, Q, UNI>;
  else return nullptr;
}

#define CB_WIN_INST(R, M, MODE, Q, UNI)                                                     \
  {R, M, MODE, Q, UNI, win_max_threads<MODE>(),                  \
   win_planes(R, Q, MODE) * win_lines(MODE), (const void *)&k_win<R, M, MODE, Q, UNI>, \
   win_batched<R, M, MODE, Q, UNI>()}
#define CB_WIN_U(R, M, MODE, U) \
  CB_WIN_INST(R, M, MODE, 0, U), CB_WIN_INST(R, M, MODE, 2, U), CB_WIN_INST(R, M, MODE, 3, U)
#define CB_WIN_ROWS_INST(R, M, MODE, Q)                                                       \
  {R, M, MODE, Q, false, win_rows_threads<MODE>(), win_planes(R, Q, MODE) * 2, \
   (const void *)&k_win_rows<R, M, MODE, Q>, nullptr}
#define CB_WIN_ROWS(R, M, MODE) \
  CB_WIN_ROWS_INST(R, M, MODE, 0), CB_WIN_ROWS_INST(R, M, MODE, 2), CB_WIN_ROWS_INST(R, M, MODE, 3)
#define CB_WIN_X(R, M) CB_WIN_U(R, M, MODE_X, true)
// the stencil by itself on unit-stride lines, in lanes of 16 rows
#define CB_WIN_STENCIL(Q)                                                                              \
  WinKernel {                                                                                          \
    1, 16, MODE_X, Q, true, win_max_threads<MODE_X>(), win_planes(1, Q, MODE_X),             \
        (const void *)&k_win<1, 16, MODE_X, Q, true, WIN_STENCIL>, nullptr              \
  }
#define CB_WIN_S(R, M) CB_WIN_U(R, M, MODE_S, false), CB_WIN_U(R, M, MODE_S, true)

}  // namespace cb
