// The two inverses of the reduced system of lanes with coefficients of their own
// (winplan.h): block elimination agrees with elimination among all rows, or says
// that it lost digits.  Prints "ok" or "BAD" and the counts.
#include <cstdio>
#include <random>

#include "../paper_2101_02286_amd/csrc/winplan.h"

using namespace cb;
using namespace cb::window;

int main() {
  std::mt19937_64 gen(7);
  std::uniform_real_distribution<double> u(-1, 1);
  int kept = 0, lost = 0, bad = 0;
  for (int t = 0; t < 600; ++t) {
    const int R = 1 + t % 3, L = t % 5 == 0 ? 2 + t % 3 : 2 + (int)(gen() % 40);
    // dominant blocks, weak ones, and ones coupled to one side alone (a cyclic
    // matrix with a good inverse whose leading blocks have none)
    const int kind = t % 4;
    BlockRing a{L, R, t % 2 == 0, std::vector<Blk>(L), std::vector<Blk>(L), std::vector<Blk>(L)};
    for (int l = 0; l < L; ++l)
      for (int q = 0; q < R * R; ++q) {
        const double diag = q / R == q % R ? 1.0 : 0.0;
        const double side = kind == 0 ? 0.1 : (kind == 1 ? 0.5 : 0.05);
        a.lo[l].v[q] = side * u(gen) + (kind >= 2 ? 1.5 * diag : 0.0);
        a.di[l].v[q] = diag * (kind == 3 ? 0.3 : 1.0) + 0.1 * u(gen);
        a.up[l].v[q] = side * u(gen);
        if (!a.cyclic && l == 0) a.lo[l].v[q] = 0.0;
        if (!a.cyclic && l == L - 1) a.up[l].v[q] = 0.0;
      }
    std::vector<double> x, y;
    if (!invert_dense(a, y)) continue;
    const bool done = R == 1 ? invert_blocks<1>(a, x) : (R == 2 ? invert_blocks<2>(a, x) : invert_blocks<3>(a, x));
    double err = 0.0, top = 0.0;
    for (size_t i = 0; i < y.size(); ++i) {
      top = std::max(top, std::fabs(y[i]));
      if (done) err = std::max(err, std::fabs(x[i] - y[i]));
    }
    if (!std::isfinite(top) || top > 1e3) continue;  // ill-conditioned, and no layout
    (done ? kept : lost) += 1;
    // both residuals are below 2^-46 or so of a row, times an inverse of 3L entries
    if (done && !(err <= std::ldexp(1.0, -45) * 3 * L * top)) {
      ++bad;
      printf("R%d L%d kind%d cyclic%d err %.2g of %.2g\n", R, L, kind, a.cyclic, err, top);
    }
  }
  printf("%s kept %d lost %d\n", bad ? "BAD" : "ok", kept, lost);
  return bad != 0;
}
