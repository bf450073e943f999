// The library's launch code and windowed-lane kernels on the host (one thread
// per work item, AddressSanitizer over exact-size buffers and LDS), through the
// C ABI, against the oracle.  Reads one case per line:
//   r n axis d0 d1 pitch cyclic halfwidth precision in_place partitions batch
// (cyclic: + 2 for bands that vary by row; d0, d1: the other extents in axis order; pitch: spare elements per x row;
// halfwidth 0: plain solve; r = 0: the stencil by itself) and prints "ok" or "BAD", whether a windowed kernel
// ran, and the relative error.
#include <hip/hip_runtime.h>
#include <pthread.h>
#include <sanitizer/asan_interface.h>

#include <cmath>
#include <cstdio>
#include <random>
#include <thread>
#include <vector>

#include "../paper_2101_02286_amd/csrc/win.h"

extern "C" int orc_solve_lines(int r, int n, const double *bands, int per_row, int cyclic, int64_t nlines,
                               const double *b, double *x);
thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;

namespace cb {
alignas(256) double smem[163840 / sizeof(double)];

// the instances that the cases use
static const WinKernel kTable[] = {
    CB_WIN_X(1, 8), CB_WIN_X(1, 10), CB_WIN_X(1, 12),
    CB_WIN_X(1, 16), CB_WIN_X(2, 16), CB_WIN_X(2, 20),
    CB_WIN_X(2, 24), CB_WIN_S(1, 8),  CB_WIN_S(2, 8),
    CB_WIN_S(2, 12), CB_WIN_S(2, 16), CB_WIN_S(1, 16),
};
const WinKernel *find_win_kernel(int R, int M, int mode, int Q, bool uni) {
  for (const auto &k : kTable)
    if (k.R == R && k.M == M && k.mode == mode && k.Q == Q && k.uni == uni) return &k;
  return nullptr;
}
const WinKernel *find_win_rows_kernel(int R, int M, int mode, int Q) {
  static const WinKernel t[] = {CB_WIN_ROWS(1, 8, MODE_X),  CB_WIN_ROWS(1, 12, MODE_X), CB_WIN_ROWS(1, 16, MODE_X),
                                CB_WIN_ROWS(2, 8, MODE_X),  CB_WIN_ROWS(2, 12, MODE_X), CB_WIN_ROWS(2, 16, MODE_X), CB_WIN_ROWS(3, 16, MODE_X),
                                CB_WIN_ROWS(1, 12, MODE_S), CB_WIN_ROWS(1, 16, MODE_S), CB_WIN_ROWS(2, 8, MODE_S),
                                CB_WIN_ROWS(2, 16, MODE_S), CB_WIN_ROWS(3, 12, MODE_S)};
  for (const auto &k : t)
    if (k.R == R && k.M == M && k.mode == mode && k.Q == Q) return &k;
  return nullptr;
}
// anything else is named but not run
const WinKernel *find_win_copy_kernel(int, int, bool) { return nullptr; }
const LineKernel *find_line_kernel(int, int, int, int, int, bool, bool) {
  static const LineKernel k{1, 1, 0, 0, 0, false, false, 1024, nullptr};
  return &k;
}
const LineKernel *find_copy_kernel(int, int, bool) { return nullptr; }
const BatchKernel *find_batch_kernel(int, int, int, bool, bool, int, int) { return nullptr; }
const WgKernel *find_wg_kernel(int, int, int, int, bool) {
  static const WgKernel k{1, 1, 0, 0, false, 1024};
  return &k;
}
const WgKernel *find_wg32_kernel(int, int, int, int, bool) { return nullptr; }
const void *stencil_kernel(int) { return nullptr; }
const WinKernel *find_win_stencil_kernel(int Q) {
  static const WinKernel k[2] = {CB_WIN_STENCIL(2), CB_WIN_STENCIL(3)};
  return &k[Q > 2 ? 1 : 0];
}
}  // namespace cb

static pthread_barrier_t g_block;
static std::vector<pthread_barrier_t> g_wave;
static int g_windowed = 0;
void host_block_barrier() { pthread_barrier_wait(&g_block); }
void host_wave_barrier() { pthread_barrier_wait(&g_wave[threadIdx.x / 64]); }

hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t) {
  if (!fn) return hipSuccess;
  bool batched = false;
  for (const auto &k : cb::kTable) batched = batched || fn == k.batch_fn;
  ++g_windowed;
  for (double &v : cb::smem) v = 1e300;  // what nobody wrote must not be read
  const size_t used = (lds + 7) / 8 * 8;
  __asan_poison_memory_region(reinterpret_cast<char *>(cb::smem) + used, sizeof(cb::smem) - used);
  g_wave.resize(block.x / 64);
  pthread_barrier_init(&g_block, nullptr, block.x);
  for (auto &w : g_wave) pthread_barrier_init(&w, nullptr, 64);
  std::vector<std::thread> th;
  for (unsigned t = 0; t < block.x; ++t)
    th.emplace_back([=] {
      threadIdx = dim3(t);
      blockDim = block;
      gridDim = grid;
      for (unsigned b = 0; b < grid.x; ++b) {
        blockIdx = dim3(b);
        if (batched)
          reinterpret_cast<void (*)(cb::BatchHdr *, const cb::WinItemDev *, int)>(const_cast<void *>(fn))(
              *static_cast<cb::BatchHdr **>(args[0]), *static_cast<const cb::WinItemDev **>(args[1]), 0);
        else
          reinterpret_cast<void (*)(cb::WinArgs)>(const_cast<void *>(fn))(*static_cast<cb::WinArgs *>(args[0]));
        host_block_barrier();
      }
    });
  for (auto &t : th) t.join();
  __asan_unpoison_memory_region(cb::smem, sizeof(cb::smem));
  return hipSuccess;
}

int main() {
  static const std::vector<double> kBands[4] = {
      {}, {1 / 3., 1, 1 / 3.}, {.05, .5, 1, .5, .05}, {1 / 400., .09, .5625, 1, .5625, .09, 1 / 400.}};
  int bad = 0, r, n, axis, d0, d1, pitch, cyclic, half, prec, in_place, parts, batch;
  while (scanf("%d %d %d %d %d %d %d %d %d %d %d %d", &r, &n, &axis, &d0, &d1, &pitch, &cyclic, &half, &prec, &in_place,
               &parts, &batch) == 12) {
    cb_plan_desc d = {};
    d.r = r;
    d.n = n;
    const bool rows = cyclic >= 2;
    cyclic &= 1;
    std::vector<double> bands = kBands[r];
    if (rows) {
      std::mt19937_64 gen(7 * n + r);
      std::uniform_real_distribution<double> u(0.5, 1.5);
      bands.clear();
      for (int j = 0; j < n; ++j)
        for (double v : kBands[r]) bands.push_back(v * u(gen) * (v == 1 ? 2 : 1));
    }
    d.bands = bands.data();
    d.per_row = rows;
    d.cyclic = cyclic;
    d.precision = prec;
    d.partitions = parts;
    cb_plan_t p = nullptr;
    if (r && cb_plan(&d, &p) != CB_OK) return printf("plan: %s\n", cb_last_error()), 1;
    cb_grid g;
    const int other[2] = {d0, d1};
    for (int i = 0, k = 0; i < 3; ++i) g.n[i] = i == axis ? n : other[k++];
    g.stride[0] = 1;
    g.stride[1] = g.n[0] + pitch;
    g.stride[2] = g.stride[1] * g.n[1];
    // exactly the elements that the grid spans
    const size_t span = (size_t)((g.n[0] - 1) + (g.n[1] - 1) * g.stride[1] + (g.n[2] - 1) * g.stride[2] + 1);
    double *in = new double[span], *out = in_place ? in : new double[span];
    std::mt19937_64 gen(n + r);
    std::uniform_real_distribution<double> u(-1, 1);
    for (size_t i = 0; i < span; ++i) in[i] = u(gen);
    std::vector<double> b0(in, in + span);
    if (!in_place)
      for (size_t i = 0; i < span; ++i) out[i] = 7.0;
    cb_stencil st = {-half, half, {}};
    for (int q = 0; q <= 2 * half && half; ++q) st.coef[q] = 0.3 * (q - half) + 0.1 * (q == half);
    g_windowed = 0;
    cb_status s;
    if (!r) {
      s = cb_rhs_stencil(&st, &g, axis, in, out, nullptr);
    } else if (batch) {
      cb_batch_item it = {p, half ? &st : nullptr, g, axis, in, out};
      std::vector<char> ws(cb_batch_workspace_bytes(&it, 1));
      s = cb_solve_batched(&it, 1, ws.data(), ws.size(), 1, nullptr);
    } else {
      s = half ? cb_apply_derivative(p, &st, &g, axis, in, out, nullptr) : cb_solve(p, &g, axis, in, out, nullptr);
    }
    const bool ran = g_windowed > 0;
    double err = 0, top = 0;
    std::vector<char> inside(span, 0);
    std::vector<double> rhs(n), x(n);
    const int ua = axis == 0 ? 1 : 0, va = axis == 2 ? 1 : 2;
    for (int64_t v = 0; v < g.n[va]; ++v)
      for (int64_t w = 0; w < g.n[ua]; ++w) {
        const int64_t base = v * g.stride[va] + w * g.stride[ua];
        for (int j = 0; j < n; ++j) {
          rhs[j] = half ? 0.0 : b0[base + j * g.stride[axis]];
          for (int q = -half; q <= half && half; ++q)
            rhs[j] += st.coef[q + half] * b0[base + ((j + q + n) % n) * g.stride[axis]];
        }
        x = rhs;
        if (r) orc_solve_lines(r, n, bands.data(), rows, cyclic, 1, rhs.data(), x.data());
        for (int j = 0; j < n; ++j) {
          const int64_t at = base + j * g.stride[axis];
          inside[at] = 1;
          err = std::fmax(err, std::isfinite(out[at]) ? std::fabs(out[at] - x[j]) : INFINITY);
          top = std::fmax(top, std::fabs(x[j]));
        }
      }
    bool ok = s == CB_OK && (!ran || err <= (prec == CB_FP32 ? 3e-6 : 1e-12) * top);
    for (size_t i = 0; i < span; ++i) ok = ok && (inside[i] || out[i] == (in_place ? b0[i] : 7.0));  // no stray stores
    printf("%s windowed=%d err=%.2g: r%d n%d axis%d %dx%d+%d rows%d cyclic%d half%d prec%d in_place%d parts%d batch%d\n",
           ok ? "ok" : "BAD", ran, err / top, r, n, axis, d0, d1, pitch, rows, cyclic, half, prec, in_place, parts, batch);
    fflush(stdout);
    bad += !ok;
    if (r) cb_plan_destroy(p);
    delete[] in;
    if (!in_place) delete[] out;
  }
  return bad != 0;
}
