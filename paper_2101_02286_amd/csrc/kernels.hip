// HIP kernels of libcb for gfx950 (MI355X): the FP64 instances of the
// two-level (P > 1) kernels (wg.h), the standalone stencil, and the dispatch
// to the line and batched kernels.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>

#include "device.h"
#include "launch.h"
#include "line.h"
#include "wg.h"
#include "win.h"

namespace cb {

// ------------------------------------------------------------------------
// Standalone periodic stencil b = sum_q c_q f_{j+q} along one axis: bound by
// HBM (16 B per point).  Each value is read from memory once and from the
// caches, LDS or registers for its other taps; the taps add up in order of q.
// Unit-stride lines go through the LDS tile of the windowed lanes (win.h):
// direct 16-byte loads of every tap ran at 2.4-3.7 TB/s, bound by the address
// unit, against 5.3-5.9.  Sixth-order weights, one 256 x 200 x 384 pass along x
// and y each: one point per thread and 64-bit divisions 136 us, now 54 and 64.
// ------------------------------------------------------------------------
typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));  // any 8-byte address

static const WinKernel kWinStencil[] = {CB_WIN_STENCIL(2), CB_WIN_STENCIL(3)};
const WinKernel *find_win_stencil_kernel(int Q) { return &kWinStencil[Q > 2 ? 1 : 0]; }

__device__ __forceinline__ int wrap_row(int j, int n) {
  while (j < 0) j += n;
  while (j >= n) j -= n;
  return j;
}

// Strided lines that lie next to each other: a wavefront takes 64 pairs of
// adjacent lines and kRows rows of them, of which it keeps the last seven in
// registers (row addresses are the same for all its threads).  8 rows measured
// 2-7 % faster than 16 on rows that are whole cache lines, up to 10 % slower on
// others, which gain more from rows that stay close in time.
template <int kRows>
__global__ __launch_bounds__(256) void k_stencil_s(const StencilArgs a) {
  const FastDiv fq{a.dq.d, a.dq.mul, a.dq.s1, a.dq.s2}, fu{a.du.d, a.du.mul, a.du.s1, a.du.s2};
  uint32_t tile = blockIdx.x;
  if (a.xcds > 1) {  // neighbouring tiles share rows: on one XCD, as in k_line
    const uint32_t X = (uint32_t)a.xcds, G = gridDim.x, q = G / X, rem = G % X, x = tile % X, s = tile / X;
    tile = x * q + (x < rem ? x : rem) + s;
  }
  // tile -> (run of 64 pairs of lines, 4 runs of rows)
  const uint32_t rest = fq.div(tile), pt = tile - rest * a.dq.d;
  const uint32_t v = fu.div(rest), jt = rest - v * a.du.d;
  const int n = (int)a.n;
  const int j0 = __builtin_amdgcn_readfirstlane(((int)jt * 4 + (int)(threadIdx.x >> 6)) * kRows);
  const uint32_t u = 2 * (pt * 64 + (threadIdx.x & 63));
  if (j0 >= n || u >= (uint32_t)a.nu) return;
  const bool one = u + 1 == (uint32_t)a.nu;
  const int64_t base = (int64_t)u + (int64_t)v * a.sv;
  const double *f = a.f + base;
  double *b = a.b + base;
  auto load = [&](int j) -> dbl2u {
    const double *p = f + (int64_t)wrap_row(j, n) * a.rs;
    if (one) return dbl2u{*p, 0.0};
    return *reinterpret_cast<const dbl2u *>(p);
  };
  dbl2u w[7];
#pragma unroll
  for (int q = -3; q < 3; ++q) w[q + 3] = q >= a.lo && q < a.hi ? load(j0 + q) : dbl2u{0.0, 0.0};
#pragma unroll
  for (int k = 0; k < kRows; ++k) {
    if (j0 + k >= n) break;
    // the row that enters: the highest tap's
    const dbl2u next = load(j0 + k + a.hi);
#pragma unroll
    for (int q = -3; q <= 3; ++q)
      if (q == a.hi) w[q + 3] = next;
    dbl2u acc = {0.0, 0.0};
#pragma unroll
    for (int q = -3; q <= 3; ++q)
      if (q >= a.lo && q <= a.hi) acc += a.c[q - a.lo] * w[q + 3];
    double *p = b + (int64_t)(j0 + k) * a.rs;
    if (one) *p = acc.x;
    else if (a.nt) __builtin_nontemporal_store(acc, reinterpret_cast<dbl2u *>(p));
    else *reinterpret_cast<dbl2u *>(p) = acc;
#pragma unroll
    for (int q = 0; q < 6; ++q) w[q] = w[q + 1];
  }
}

// Any positive strides and any size: small fields, narrow rows and short lines.
// TINY: lines shorter than the stencil's reach, whose taps wrap more than once (a
// check of that in the one instance cost 5 %).
template <bool TINY>
__global__ __launch_bounds__(256) void k_stencil(const StencilArgs a) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= a.total) return;
  // consecutive threads touch consecutive addresses: along the line when it
  // is unit-stride (idx = (v, u, j)), else across lines (idx = (v, j, u))
  int64_t u, j, vv;
  if (a.rs == 1) {
    j = idx % a.n;
    const int64_t rest = idx / a.n;
    u = rest % a.nu;
    vv = rest / a.nu;
  } else {
    u = idx % a.nu;
    const int64_t rest = idx / a.nu;
    j = rest % a.n;
    vv = rest / a.n;
  }
  const int64_t base = u * a.su + vv * a.sv;
  double acc = 0.0;
  for (int q = a.lo; q <= a.hi; ++q) {
    int64_t jj = j + q;
    if (TINY) jj = (jj + 3 * a.n) % a.n;
    else jj = jj < 0 ? jj + a.n : (jj >= a.n ? jj - a.n : jj);
    acc += a.c[q - a.lo] * a.f[base + jj * a.rs];
  }
  a.b[base + j * a.rs] = acc;
}

// ------------------------------------------------------------------------
// Dispatch tables
// ------------------------------------------------------------------------
const LineKernel *find_line_kernel(int R, int M, int fp32, int mode, int Q, bool uni, bool ilu) {
  int cnt = 0;
  const LineKernel *t = nullptr;
  if (R == 3) {
    if (M == 8) t = line_table_r3_m8(&cnt);
    else if (M == 16) t = line_table_r3_m16(&cnt);
    else return nullptr;
  } else switch (M) {
    case 4: t = line_table_m4(&cnt); break;
    case 6: t = line_table_m6(&cnt); break;
    case 8: t = line_table_m8(&cnt); break;
    case 12: t = line_table_m12(&cnt); break;
    case 16: t = line_table_m16(&cnt); break;
    case 32: t = line_table_m32(&cnt); break;
    default: return nullptr;
  }
  for (int i = 0; i < cnt; ++i)
    if (t[i].R == R && t[i].M == M && t[i].fp32 == fp32 && t[i].mode == mode && t[i].Q == Q && t[i].uni == uni &&
        t[i].ilu == ilu)
      return &t[i];
  return nullptr;
}

#define CB_WG_INST(R, M, MODE, Q, ILU)                                                                 \
  {R, M, MODE, Q, ILU, wg_max_threads<M, MODE>(), (const void *)&k_wg_a<R, MODE, Q>,                      \
   (const void *)&k_wg_b<R>, (const void *)&k_wg_c<R, M, MODE, Q, ILU>, nullptr, nullptr, nullptr,        \
   ILU ? (const void *)&k_wg_c<R, M, MODE, Q, true, double, false, true> : nullptr}
#define CB_WG_I(R, M, MODE, Q) CB_WG_INST(R, M, MODE, Q, false), CB_WG_INST(R, M, MODE, Q, true)
#define CB_WG_Q(R, M, MODE) CB_WG_I(R, M, MODE, 0), CB_WG_I(R, M, MODE, 2), CB_WG_I(R, M, MODE, 3)
static const WgKernel kWgKernels[] = {
    CB_WG_Q(1, 8, MODE_X), CB_WG_Q(1, 8, MODE_S), CB_WG_Q(2, 8, MODE_X), CB_WG_Q(2, 8, MODE_S),
    CB_WG_Q(1, 16, MODE_X), CB_WG_Q(1, 16, MODE_S), CB_WG_Q(2, 16, MODE_X), CB_WG_Q(2, 16, MODE_S),
    CB_WG_Q(3, 8, MODE_X),  CB_WG_Q(3, 8, MODE_S),  CB_WG_Q(3, 16, MODE_X), CB_WG_Q(3, 16, MODE_S),
};

const WgKernel *find_wg_kernel(int R, int M, int mode, int Q, bool ilu) {
  for (const auto &k : kWgKernels)
    if (k.R == R && k.M == M && k.mode == mode && k.Q == Q && k.ilu == ilu) return &k;
  return nullptr;
}

const WgKernel *wg32_table_m8(int *count);
const WgKernel *wg32_table_m16(int *count);

const WgKernel *find_wg32_kernel(int R, int M, int mode, int Q, bool ilu) {
  int cnt = 0;
  const WgKernel *t = M == 8 ? wg32_table_m8(&cnt) : (M == 16 ? wg32_table_m16(&cnt) : nullptr);
  for (int i = 0; i < cnt; ++i)
    if (t[i].R == R && t[i].M == M && t[i].mode == mode && t[i].Q == Q && t[i].ilu == ilu) return &t[i];
  return nullptr;
}

const WinKernel *win_table_r1_x(int *count);
const WinKernel *win_table_r1_s(int *count);
const WinKernel *win_table_r2_x(int *count);
const WinKernel *win_table_r2_s(int *count);
const WinKernel *win_table_r3_x(int *count);
const WinKernel *win_table_r3_s(int *count);

const WinKernel *win_table_rows_r1(int *count);
const WinKernel *win_table_rows_r2(int *count);
const WinKernel *win_table_rows_r3(int *count);

const WinKernel *find_win_rows_kernel(int R, int M, int mode, int Q) {
  int cnt = 0;
  const WinKernel *t = R == 1 ? win_table_rows_r1(&cnt) : (R == 2 ? win_table_rows_r2(&cnt) : win_table_rows_r3(&cnt));
  for (int i = 0; i < cnt; ++i)
    if (t[i].M == M && t[i].mode == mode && t[i].Q == Q) return &t[i];
  return nullptr;
}

const WinKernel *find_win_kernel(int R, int M, int mode, int Q, bool uni) {
  const WinKernel *(*const tables[])(int *) = {win_table_r1_x, win_table_r1_s, win_table_r2_x, win_table_r2_s,
                                              win_table_r3_x, win_table_r3_s};
  for (auto table : tables) {
    int cnt = 0;
    const WinKernel *t = table(&cnt);
    if (t[0].R != R || t[0].mode != mode) continue;
    for (int i = 0; i < cnt; ++i)
      if (t[i].R == R && t[i].M == M && t[i].mode == mode && t[i].Q == Q && t[i].uni == uni)
        return &t[i];
  }
  return nullptr;
}

const void *stencil_kernel(int form) {
  return form == STENCIL_S         ? (const void *)&k_stencil_s<kStencilRows>
         : form == STENCIL_S_SHORT ? (const void *)&k_stencil_s<kStencilRows / 2>
         : form == STENCIL_TINY    ? (const void *)&k_stencil<true>
                                   : (const void *)&k_stencil<false>;
}

const BatchKernel *find_batch_kernel(int R, int M, int fp32, bool uni, bool ilu, int mode, int Q) {
  int cnt = 0;
  const BatchKernel *t = nullptr;
  if (R == 3) {
    if (M == 8) t = batch_table_r3_m8(&cnt);
    else if (M == 16) t = batch_table_r3_m16(&cnt);
    else return nullptr;
  } else switch (M) {
    case 4: t = batch_table_m4(&cnt); break;
    case 6: t = batch_table_m6(&cnt); break;
    case 8: t = batch_table_m8(&cnt); break;
    case 12: t = batch_table_m12(&cnt); break;
    case 16: t = batch_table_m16(&cnt); break;
    case 32: t = batch_table_m32(&cnt); break;
    default: return nullptr;
  }
  for (int i = 0; i < cnt; ++i)
    if (t[i].R == R && t[i].M == M && t[i].fp32 == fp32 && t[i].uni == uni && t[i].ilu == ilu && t[i].mode == mode &&
        t[i].Q == Q)
      return &t[i];
  return nullptr;
}

}  // namespace cb
