// Windowed-lane launches on the host with LDS that holds NaN until a workgroup
// writes it, so that a slot read before it is written shows in the results even
// behind a zero coefficient; and batches of several items in either form, with
// the wavefronts that leave a workgroup early.  The library's kernels, runtime
// stand-ins and oracle are those of windowed_host.cpp.  Reads one launch per line:
//   form items, then for each item: r n axis d0 d1 cyclic halfwidth
// (form 0: single calls; 1: a batch with a workgroup per tile; 2: a batch on the
// persistent queue; d0, d1: the other extents in axis order; cyclic: + 2 for bands
// that vary by row, with the first half of the rows and of the right-hand side
// scaled by 2^-9; halfwidth 0: plain solve) and prints "ok" or "BAD", the windowed launches and the largest
// relative error.
#include <hip/hip_runtime.h>
#define main main_of_single_calls
#define hipLaunchKernel launch_of_single_calls
#define host_block_barrier barrier_of_single_calls
#define find_win_kernel find_win_kernel_of_single_calls
#define find_win_rows_kernel find_win_rows_kernel_of_single_calls
#include "windowed_host.cpp"
#undef main
#undef hipLaunchKernel
#undef host_block_barrier
#undef find_win_kernel
#undef find_win_rows_kernel

#include <condition_variable>
#include <limits>
#include <mutex>

// (built without the sanitizer that windowed_host.cpp runs under)
extern "C" void __asan_poison_memory_region(const volatile void *, size_t) {}
extern "C" void __asan_unpoison_memory_region(const volatile void *, size_t) {}

namespace cb {
static const WinKernel kMore[] = {CB_WIN_S(1, 12), CB_WIN_S(3, 16)};
const WinKernel *find_win_kernel(int R, int M, int mode, int Q, bool uni) {
  for (const auto &k : kMore)
    if (k.R == R && k.M == M && k.mode == mode && k.Q == Q && k.uni == uni) return &k;
  return find_win_kernel_of_single_calls(R, M, mode, Q, uni);
}
const WinKernel *find_win_rows_kernel(int R, int M, int mode, int Q) {
  static const WinKernel k[] = {CB_WIN_ROWS(1, 8, MODE_S)};
  return R == 1 && M == 8 && mode == MODE_S ? &k[Q ? Q - 1 : 0] : find_win_rows_kernel_of_single_calls(R, M, mode, Q);
}
}  // namespace cb

// A workgroup's barrier counts the wavefronts that have not left.
static std::mutex g_mu;
static std::condition_variable g_cv;
static unsigned g_live, g_waiting, g_round;
static void release() {
  g_waiting = 0;
  ++g_round;
  g_cv.notify_all();
}
void host_block_barrier() {
  std::unique_lock<std::mutex> lk(g_mu);
  const unsigned round = g_round;
  if (++g_waiting == g_live) return release();
  g_cv.wait(lk, [&] { return g_round != round; });
}
static void leave() {
  std::lock_guard<std::mutex> lk(g_mu);
  --g_live;
  if (g_live && g_waiting == g_live) release();
}

hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t) {
  if (!fn) return hipSuccess;
  bool batched = false;
  for (const auto &k : cb::kTable) batched = batched || fn == k.batch_fn;
  for (const auto &k : cb::kMore) batched = batched || fn == k.batch_fn;
  ++g_windowed;
  const size_t used = (lds + 7) / 8 * 8;
  g_wave.resize(block.x / 64);
  for (auto &w : g_wave) pthread_barrier_init(&w, nullptr, 64);
  pthread_barrier_t all;
  pthread_barrier_init(&all, nullptr, block.x);
  std::vector<std::thread> th;
  for (unsigned t = 0; t < block.x; ++t)
    th.emplace_back([=, &all] {
      threadIdx = dim3(t);
      blockDim = block;
      gridDim = grid;
      for (unsigned b = 0; b < grid.x; ++b) {
        blockIdx = dim3(b);
        if (t == 0) {
          std::fill_n(cb::smem, used / 8, std::numeric_limits<double>::quiet_NaN());
          g_live = block.x;
          g_waiting = 0;
        }
        pthread_barrier_wait(&all);
        if (batched)
          reinterpret_cast<void (*)(cb::BatchHdr *, const cb::WinItemDev *, int)>(const_cast<void *>(fn))(
              *static_cast<cb::BatchHdr **>(args[0]), *static_cast<const cb::WinItemDev **>(args[1]),
              *static_cast<int *>(args[2]));
        else
          reinterpret_cast<void (*)(cb::WinArgs)>(const_cast<void *>(fn))(*static_cast<cb::WinArgs *>(args[0]));
        leave();
        pthread_barrier_wait(&all);
      }
    });
  for (auto &t : th) t.join();
  pthread_barrier_destroy(&all);
  for (auto &w : g_wave) pthread_barrier_destroy(&w);
  return hipSuccess;
}

struct Item {
  int r, n, axis, cyclic, half;
  bool rows;
  cb_plan_t plan = nullptr;
  cb_stencil st{};
  cb_grid g{};
  std::vector<double> bands, in, out;
};

// Largest error of an item's lines over the largest value (infinite when one is not finite).
static double error_of(const Item &it) {
  double err = 0, top = 0;
  std::vector<double> rhs(it.n), x(it.n);
  const int ua = it.axis == 0 ? 1 : 0, va = it.axis == 2 ? 1 : 2;
  for (int64_t v = 0; v < it.g.n[va]; ++v)
    for (int64_t u = 0; u < it.g.n[ua]; ++u) {
      const int64_t base = v * it.g.stride[va] + u * it.g.stride[ua], rs = it.g.stride[it.axis];
      for (int j = 0; j < it.n; ++j) {
        rhs[j] = it.half ? 0.0 : it.in[base + j * rs];
        for (int q = -it.half; q <= it.half && it.half; ++q)
          rhs[j] += it.st.coef[q + it.half] * it.in[base + ((j + q + it.n) % it.n) * rs];
      }
      orc_solve_lines(it.r, it.n, it.bands.data(), it.rows, it.cyclic, 1, rhs.data(), x.data());
      for (int j = 0; j < it.n; ++j) {
        const double o = it.out[base + j * rs];
        err = std::fmax(err, std::isfinite(o) ? std::fabs(o - x[j]) : INFINITY);
        top = std::fmax(top, std::fabs(x[j]));
      }
    }
  return err / top;
}

int main() {
  static const std::vector<double> kBands[4] = {
      {}, {1 / 3., 1, 1 / 3.}, {.05, .5, 1, .5, .05}, {1 / 400., .09, .5625, 1, .5625, .09, 1 / 400.}};
  int bad = 0, form, count;
  while (scanf("%d %d", &form, &count) == 2) {
    std::vector<Item> items(count);
    std::vector<cb_batch_item> list;
    for (Item &it : items) {
      int d[2];
      if (scanf("%d %d %d %d %d %d %d", &it.r, &it.n, &it.axis, &d[0], &d[1], &it.cyclic, &it.half) != 7) return 2;
      it.rows = it.cyclic >= 2;
      it.cyclic &= 1;
      it.bands.clear();
      for (int j = 0; j < (it.rows ? it.n : 1); ++j)
        for (double v : kBands[it.r]) it.bands.push_back(it.rows && j < it.n / 2 ? std::ldexp(v, -9) : v);
      cb_plan_desc desc = {};
      desc.per_row = it.rows;
      desc.r = it.r;
      desc.n = it.n;
      desc.bands = it.bands.data();
      desc.cyclic = it.cyclic;
      if (cb_plan(&desc, &it.plan) != CB_OK) return printf("plan: %s\n", cb_last_error()), 2;
      for (int i = 0, k = 0; i < 3; ++i) it.g.n[i] = i == it.axis ? it.n : d[k++];
      it.g.stride[0] = 1;
      it.g.stride[1] = it.g.n[0];
      it.g.stride[2] = it.g.n[0] * it.g.n[1];
      it.in.resize(it.g.stride[2] * it.g.n[2]);
      std::mt19937_64 gen(it.n + it.r);
      std::uniform_real_distribution<double> u(-1, 1);
      for (size_t i = 0; i < it.in.size(); ++i) {
        const int j = (int)(i / it.g.stride[it.axis] % it.n);
        it.in[i] = it.rows && j < it.n / 2 ? std::ldexp(u(gen), -9) : u(gen);
      }
      it.out.assign(it.in.size(), 7.0);
      it.st.lo = -it.half;
      it.st.hi = it.half;
      for (int q = 0; q <= 2 * it.half && it.half; ++q) it.st.coef[q] = 0.3 * (q - it.half) + 0.1 * (q == it.half);
      list.push_back({it.plan, it.half ? &it.st : nullptr, it.g, it.axis, it.in.data(), it.out.data()});
    }
    g_windowed = 0;
    cb_status s = CB_OK;
    if (form) {
      std::vector<char> ws(cb_batch_workspace_bytes(list.data(), count));
      s = cb_solve_batched(list.data(), count, ws.data(), ws.size(), form == 1 ? -1 : 1, nullptr);
    } else {
      for (const cb_batch_item &b : list)
        if (!s)
          s = b.stencil ? cb_apply_derivative(b.plan, b.stencil, &b.grid, b.axis, b.in, b.out, nullptr)
                        : cb_solve(b.plan, &b.grid, b.axis, b.in, b.out, nullptr);
    }
    const int ran = g_windowed;
    double err = 0, tol = 1e-12;  // the library's FP64 bound; for scaled rows what rounding makes of them
    for (const Item &it : items) {
      err = std::fmax(err, error_of(it));
      tol = it.rows ? 2e-14 : tol;  // 64 roundings a row of 2^-53, an inverse of norm 3
    }
    const bool ok = s == CB_OK && err <= tol;
    printf("%s windowed=%d err=%.2g: form%d r%d axis%d n", ok ? "ok" : "BAD", ran, err, form, items[0].r, items[0].axis);
    for (const Item &it : items) {
      printf(" %d", it.n);
      cb_plan_destroy(it.plan);
    }
    printf("\n");
    fflush(stdout);
    bad += !ok;
  }
  return bad != 0;
}
