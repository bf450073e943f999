// Host factorisation of windowed lanes (WinLayout in plan.h): one elimination
// of the Toeplitz band for every lane's interior block, and the windows of the
// reduced system's inverse (Sec. 3-4 with lanes as partitions).  Part of
// plan.cpp.
#pragma once
#include <algorithm>
#include <cmath>
#include <map>

#include "plan.h"

namespace cb {
namespace window {

struct Blk {  // R x R, row-major
  double v[kMaxR * kMaxR] = {};
};

Blk mul(const Blk &a, const Blk &b, int R) {
  Blk c;
  for (int i = 0; i < R; ++i)
    for (int k = 0; k < R; ++k)
      for (int j = 0; j < R; ++j) c.v[i * R + j] += a.v[i * R + k] * b.v[k * R + j];
  return c;
}
Blk sub(const Blk &a, const Blk &b, int R) {
  Blk c;
  for (int i = 0; i < R * R; ++i) c.v[i] = a.v[i] - b.v[i];
  return c;
}
Blk neg(const Blk &a, int R) {
  Blk c;
  for (int i = 0; i < R * R; ++i) c.v[i] = -a.v[i];
  return c;
}
double abs_sum(const Blk &a, int R) {
  double s = 0.0;
  for (int i = 0; i < R * R; ++i) s += std::fabs(a.v[i]);
  return s;
}

// m x m inverse by Gauss-Jordan with partial pivoting; false when a pivot is
// below 1e-10 of the largest entry.
bool invert(int m, const double *a, double *out) {
  std::vector<double> t(a, a + (size_t)m * m);
  double amax = 0.0;
  for (double v : t) amax = std::max(amax, std::fabs(v));
  if (!(amax > 0.0) || !std::isfinite(amax)) return false;
  for (int i = 0; i < m * m; ++i) out[i] = 0.0;
  for (int i = 0; i < m; ++i) out[i * m + i] = 1.0;
  for (int k = 0; k < m; ++k) {
    int p = k;
    for (int i = k + 1; i < m; ++i)
      if (std::fabs(t[i * m + k]) > std::fabs(t[p * m + k])) p = i;
    if (!(std::fabs(t[p * m + k]) > 1e-10 * amax)) return false;
    if (p != k)
      for (int j = 0; j < m; ++j) {
        std::swap(t[k * m + j], t[p * m + j]);
        std::swap(out[k * m + j], out[p * m + j]);
      }
    const double d = 1.0 / t[k * m + k];
    for (int j = 0; j < m; ++j) {
      t[k * m + j] *= d;
      out[k * m + j] *= d;
    }
    for (int i = 0; i < m; ++i) {
      const double f = t[i * m + k];
      if (i == k || f == 0.0) continue;
      for (int j = 0; j < m; ++j) {
        t[i * m + j] -= f * t[k * m + j];
        out[i * m + j] -= f * out[k * m + j];
      }
    }
  }
  return true;
}
bool invert(const Blk &a, int R, Blk &out) { return invert(R, a.v, out.v); }

// The reduced system (Eqs. (18)-(20)) of one line: blocks of lane l from the
// sizes of l and its predecessor (0: base + 1 rows, 1: base rows).
struct Reduced {
  int R = 1, L = 0, extra = 0;
  bool cyclic = true;
  Blk Lt, Ut, Dt;
  Blk Sl[2], Rl[2], Sf[2], Rf[2];  // last and first R rows of D^{-1}L and D^{-1}U
  int type(int l) const { return extra > 0 && l < extra ? 0 : 1; }
  int wrap(int l) const { return l < 0 ? l + L : (l >= L ? l - L : l); }
  Blk lower(int l) const {
    if (!cyclic && l == 0) return Blk();
    return neg(mul(Lt, Sl[type(wrap(l - 1))], R), R);
  }
  Blk upper(int l) const {
    if (!cyclic && l == L - 1) return Blk();
    return neg(mul(Ut, Rf[type(l)], R), R);
  }
  Blk diag(int l) const {
    Blk d = sub(Dt, mul(Ut, Sf[type(l)], R), R);
    if (cyclic || l > 0) d = sub(d, mul(Lt, Rl[type(wrap(l - 1))], R), R);
    return d;
  }
};

// Row l of the inverse over lanes l-K..l+K (a line of more than 2K+1 lanes, or
// an acyclic one, whose absent lanes give zeros), by eliminating towards lane l
// from both ends of the window.
bool inverse_row(const Reduced &rs, int l, int K, std::vector<Blk> &g) {
  const int R = rs.R;
  g.assign(2 * K + 1, Blk());
  auto there = [&](int j) { return rs.cyclic || (j >= 0 && j < rs.L); };
  auto id = [&](int j) { return rs.cyclic ? rs.wrap(j) : j; };
  std::vector<Blk> wl(K + 1), wr(K + 1);  // inverses of the eliminated diagonal blocks at distance 1..K
  Blk centre = rs.diag(id(l));
  for (int side = -1; side <= 1; side += 2) {
    std::vector<Blk> &w = side < 0 ? wl : wr;
    Blk corr;
    bool have = false;
    for (int d = K; d >= 1; --d) {
      const int j = l + side * d;
      if (!there(j)) continue;
      Blk a = rs.diag(id(j));
      if (have) a = sub(a, corr, R);
      if (!invert(a, R, w[d])) return false;
      // what lane j's elimination takes from the diagonal of its neighbour towards l
      const int t = j - side;
      const Blk to = side < 0 ? rs.lower(id(t)) : rs.upper(id(t));
      const Blk from = side < 0 ? rs.upper(id(j)) : rs.lower(id(j));
      corr = mul(mul(to, w[d], R), from, R);
      have = true;
    }
    if (have) centre = sub(centre, corr, R);
  }
  if (!invert(centre, R, g[K])) return false;
  for (int side = -1; side <= 1; side += 2)
    for (int d = 1; d <= K; ++d) {
      const int j = l + side * d, t = j - side;
      if (!there(j)) break;
      const Blk c = side < 0 ? rs.lower(id(t)) : rs.upper(id(t));
      g[K + side * d] = neg(mul(mul(g[K + side * (d - 1)], c, R), (side < 0 ? wl : wr)[d], R), R);
    }
  return true;
}

// A block tridiagonal matrix of L >= 2 blocks, with corners when cyclic (lo[0]
// multiplies the last lane's unknowns, up[L-1] the first's).
struct BlockRing {
  int L, R;
  bool cyclic;
  std::vector<Blk> lo, di, up;
};

// Its inverse [L][L][R][R], by elimination among all rows: O(L^3 R^3).
bool invert_dense(const BlockRing &a, std::vector<double> &inv) {
  const int L = a.L, R = a.R, m = L * R;
  std::vector<double> t((size_t)m * m, 0.0), x((size_t)m * m);
  for (int l = 0; l < L; ++l) {
    const int lm = l > 0 ? l - 1 : L - 1, lp = l + 1 < L ? l + 1 : 0;
    for (int i = 0; i < R; ++i)
      for (int c = 0; c < R; ++c) {
        t[(size_t)(l * R + i) * m + lm * R + c] += a.lo[l].v[i * R + c];
        t[(size_t)(l * R + i) * m + l * R + c] += a.di[l].v[i * R + c];
        t[(size_t)(l * R + i) * m + lp * R + c] += a.up[l].v[i * R + c];
      }
  }
  if (!invert(m, t.data(), x.data())) return false;
  inv.resize((size_t)m * m);
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < m; ++j) inv[(((size_t)(i / R) * L + j / R) * R + i % R) * R + j % R] = x[(size_t)i * m + j];
  return true;
}

// The same by block elimination from the first block, the last being a border
// of a cyclic matrix: O(L^2 R^3), and most matrices here need no pivoting among
// blocks.  False where it loses digits (a residual above 2^-46).
template <int R>
bool invert_blocks(const BlockRing &a, std::vector<double> &inv) {
  struct Mat {
    double v[R * R];
    Mat operator*(const Mat &b) const {
      Mat c;
      for (int i = 0; i < R; ++i)
        for (int j = 0; j < R; ++j) {
          c.v[i * R + j] = 0.0;
          for (int k = 0; k < R; ++k) c.v[i * R + j] += v[i * R + k] * b.v[k * R + j];
        }
      return c;
    }
    Mat plus(const Mat &b, double f) const {
      Mat c;
      for (int i = 0; i < R * R; ++i) c.v[i] = v[i] + f * b.v[i];
      return c;
    }
  };
  const int L = a.L, last = L - 1;
  const int T = a.cyclic ? L - 1 : L;  // blocks of the tridiagonal part
  std::vector<Mat> lo(L), di(L), up(L);
  for (int i = 0; i < L; ++i)
    for (int q = 0; q < R * R; ++q) {
      lo[i].v[q] = a.lo[i].v[q];
      di[i].v[q] = a.di[i].v[q];
      up[i].v[q] = a.up[i].v[q];
    }
  const Mat zero{};
  std::vector<Mat> w(T), f(T);  // inverses of the eliminated diagonal blocks; lo w of the block before
  for (int i = 0; i < T; ++i) {
    f[i] = i > 0 ? lo[i] * w[i - 1] : zero;
    const Mat d = i > 0 ? di[i].plus(f[i] * up[i - 1], -1.0) : di[i];
    if (!invert(R, d.v, w[i].v)) return false;
  }
  std::vector<Mat> x((size_t)L * L, zero);  // columns one after the other
  auto at = [&](int i, int j) -> Mat & { return x[(size_t)j * L + i]; };
  for (int j = 0; j < T; ++j) {
    for (int i = 0; i < R; ++i) at(j, j).v[i * R + i] = 1.0;
    for (int i = j + 1; i < T; ++i) at(i, j) = zero.plus(f[i] * at(i - 1, j), -1.0);
    for (int i = T - 1; i >= 0; --i) at(i, j) = w[i] * (i + 1 < T ? at(i, j).plus(up[i] * at(i + 1, j), -1.0) : at(i, j));
  }
  if (a.cyclic) {
    std::vector<Mat> tb(T), ct(T);  // the inverse so far times the border's column; its row times the inverse
    for (int i = 0; i < T; ++i) {
      tb[i] = (at(i, 0) * lo[0]).plus(at(i, T - 1) * up[T - 1], 1.0);
      ct[i] = (lo[last] * at(T - 1, i)).plus(up[last] * at(0, i), 1.0);
    }
    const Mat schur = di[last].plus(lo[last] * tb[T - 1], -1.0).plus(up[last] * tb[0], -1.0);
    if (!invert(R, schur.v, at(last, last).v)) return false;
    for (int i = 0; i < T; ++i) {
      at(i, last) = zero.plus(tb[i] * at(last, last), -1.0);
      at(last, i) = zero.plus(at(last, last) * ct[i], -1.0);
    }
    for (int j = 0; j < T; ++j)
      for (int i = 0; i < T; ++i) at(i, j) = at(i, j).plus(at(i, last) * ct[j], -1.0);
  }
  inv.resize((size_t)L * L * R * R);
  double worst = 0.0;  // of A inv - 1
  for (int j = 0; j < L; ++j)
    for (int i = 0; i < L; ++i) {
      std::copy(at(i, j).v, at(i, j).v + R * R, inv.begin() + ((size_t)i * L + j) * R * R);
      Mat e = di[i] * at(i, j);
      if (a.cyclic || i > 0) e = e.plus(lo[i] * at(i > 0 ? i - 1 : last, j), 1.0);
      if (a.cyclic || i < last) e = e.plus(up[i] * at(i < last ? i + 1 : 0, j), 1.0);
      for (int q = 0; q < R * R; ++q) {
        const double r = std::fabs(e.v[q] - (i == j && q / R == q % R ? 1.0 : 0.0));
        worst = r <= worst ? worst : r;  // (NaN stays)
      }
    }
  return worst <= std::ldexp(1.0, -46);
}

}  // namespace window

bool build_window(int n, int R, const double *bands, bool cyclic, int M, double tol, bool ring, WinLayout &w) {
  using namespace window;
  const int W = 2 * R + 1, N = M - R;
  const int L = (n + M - 1) / M;
  if (L < 2 || N < R + 1) return false;
  ring = ring && n % M != 0;
  if (ring ? !cyclic : ((n + L - 1) / L != M || n / L < 2 * R + 1)) return false;
  w = WinLayout();
  const int base = ring ? M : n / L, extra = ring ? 0 : n % L;
  const bool two = extra > 0;  // lanes of two sizes
  auto a = [&](int o) { return o < -R || o > R ? 0.0 : bands[o + R]; };
  double scale = 0.0;
  for (int o = 0; o < W; ++o) scale = std::max(scale, std::fabs(bands[o]));
  // Toeplitz elimination of N + R rows (the rows beyond N only complete u)
  const int NE = N + R;
  std::vector<double> k((size_t)NE * R, 0.0), u((size_t)NE * R, 0.0), dinv(NE);
  {
    std::vector<double> c((size_t)NE * W, 0.0);
    for (int j = 0; j < NE; ++j)
      for (int o = -R; o <= R; ++o)
        if (j + o >= 0 && j + o < NE) c[(size_t)j * W + o + R] = a(o);
    for (int j = 0; j < NE; ++j) {
      const double piv = c[(size_t)j * W + R];
      if (!(std::fabs(piv) > 1e-2 * scale) || !std::isfinite(piv)) return false;
      dinv[j] = 1.0 / piv;
      for (int i = j + 1; i <= std::min(NE - 1, j + R); ++i) {
        const double f = c[(size_t)i * W + (j - i + R)] / piv;
        k[(size_t)i * R + (i - j) - 1] = f;
        for (int q = j + 1; q <= std::min(NE - 1, j + R); ++q) c[(size_t)i * W + (q - i + R)] -= f * c[(size_t)j * W + (q - j + R)];
      }
      for (int q = 1; q <= R; ++q) u[(size_t)j * R + q - 1] = j + q < NE ? c[(size_t)j * W + R + q] * dinv[j] : 0.0;
    }
  }
  auto forward = [&](int m, double *x) {
    for (int j = 1; j < m; ++j)
      for (int q = 1; q <= R && q <= j; ++q) x[j] -= k[(size_t)j * R + q - 1] * x[j - q];
  };
  auto backward = [&](int m, double *x) {
    for (int j = m - 1; j >= 0; --j) {
      double s = x[j] * dinv[j];
      for (int q = 1; q <= R && j + q < m; ++q) s -= u[(size_t)j * R + q - 1] * x[j + q];
      x[j] = s;
    }
  };
  Reduced rs;
  rs.R = R;
  rs.L = L;
  rs.extra = extra;
  rs.cyclic = cyclic;
  for (int i = 0; i < R; ++i)
    for (int c = 0; c < R; ++c) {
      rs.Lt.v[i * R + c] = a(c - R - i);
      rs.Dt.v[i * R + c] = a(c - i);
      rs.Ut.v[i * R + c] = a(R + c - i);
    }
  // the row table
  const int RW = win_row_size(R);
  w.coef.assign((size_t)N * RW + 2 * R * R, 0.0);
  std::vector<double> wf((size_t)R * N, 0.0);  // first R rows of U^{-1}
  for (int i = 0; i < R; ++i) {
    std::vector<double> p(N + R, 0.0);
    p[i] = 1.0;
    for (int j = i; j < N; ++j) {
      wf[(size_t)i * N + j] = p[j] * dinv[j];
      for (int q = 1; q <= R; ++q) p[j + q] -= p[j] * u[(size_t)j * R + q - 1];
    }
  }
  double biggest = 0.0;
  std::vector<double> col(N);
  for (int c = 0; c < R; ++c) {
    for (int j = 0; j < N; ++j) col[j] = a(c - R - j);
    forward(N, col.data());
    for (int j = 0; j < N; ++j) w.coef[(size_t)j * RW + 2 * R + c] = col[j];
  }
  for (int j = 0; j < N; ++j) {
    double *row = w.coef.data() + (size_t)j * RW;
    for (int q = 0; q < R; ++q) {
      row[q] = k[(size_t)j * R + q];
      row[3 * R + 1 + q] = u[(size_t)j * R + q];
      for (int i = 0; i < R; ++i) row[R + q] += rs.Ut.v[q * R + i] * wf[(size_t)i * N + j];
    }
    row[3 * R] = dinv[j];
    for (int q = 0; q < RW; ++q)  // (ell alone grows with the bands' scale)
      if (q != 3 * R) biggest = std::max(biggest, std::fabs(row[q]) / (q / R == 2 ? scale : 1.0));
  }
  if (!(biggest <= 64.0)) return false;  // elimination that grows needs pivoting
  for (int ty = 0; ty < 2; ++ty) {
    const int m = ty == 0 || !two ? N : N - 1;  // interior rows of this lane size
    // z: L~ times the last R rows of U^{-1}, on the last R values of z
    double *z = w.coef.data() + (size_t)N * RW + ty * R * R;
    for (int i = 0; i < R; ++i) {
      std::vector<double> e(m, 0.0);
      e[m - R + i] = 1.0;
      backward(m, e.data());
      for (int s = 0; s < R; ++s)
        for (int b = 0; b < R; ++b) z[b * R + i] += rs.Lt.v[b * R + s] * e[m - R + s];
    }
    for (int c = 0; c < R; ++c) {
      std::vector<double> x(m);
      for (int j = 0; j < m; ++j) x[j] = a(c - R - j);
      forward(m, x.data());
      backward(m, x.data());
      for (int s = 0; s < R; ++s) {
        rs.Sf[ty].v[s * R + c] = x[s];
        rs.Sl[ty].v[s * R + c] = x[m - R + s];
      }
      for (int j = 0; j < m; ++j) x[j] = a(m + c - j);
      forward(m, x.data());
      backward(m, x.data());
      for (int s = 0; s < R; ++s) {
        rs.Rf[ty].v[s * R + c] = x[s];
        rs.Rl[ty].v[s * R + c] = x[m - R + s];
      }
    }
  }
  // window half-width from a line of the smaller lanes (the slowest decay)
  constexpr int K0 = 2 * kWinMaxD;
  std::vector<Blk> g;
  int D = 0;
  {
    Reduced all = rs;
    all.L = 4 * K0;
    all.extra = 0;
    all.cyclic = true;
    double sum = 0.0, out = 0.0;
    bool ok = inverse_row(all, 0, K0, g);
    if (ok) {
      for (const Blk &b : g) sum += abs_sum(b, R);
      D = K0;
      while (D > 0 && out + abs_sum(g[K0 - D], R) + abs_sum(g[K0 + D], R) <= tol * sum) {
        out += abs_sum(g[K0 - D], R) + abs_sum(g[K0 + D], R);
        --D;
      }
      ok = std::isfinite(sum) && sum * scale <= 1e4;
    }
    if (!ok) D = K0;
  }
  D = std::max(D, 1);
  // a short line's window holds every lane (nothing is left out)
  const bool whole = cyclic && !ring && D >= L / 2;
  if (whole) D = std::max(1, L / 2);
  if (D > kWinMaxD) return false;
  // (nor does an acyclic line's reach further than its lanes: a launch exchanges
  // the values of L lanes, and slots beyond them hold nothing)
  if (!cyclic) D = std::min(D, L - 1);
  w.M = M;
  w.L = L;
  w.base = base;
  w.extra = extra;
  w.D = D;
  w.uniform = cyclic && !two ? 1 : 0;
  const int K = D + 3, RR = R * R;
  w.gidx.assign(L, 0);
  auto put = [&](const std::vector<Blk> &row, int centre) {
    for (int d = -D; d <= D; ++d)
      for (int q = 0; q < RR; ++q) w.g.push_back(row[centre + d].v[q]);
  };
  if (ring) {  // lanes around the line without end
    put(g, K0);
    return true;
  }
  if (cyclic && L < 2 * K + 2) {  // few lanes: the dense inverse
    BlockRing ring{L, R, true, {}, {}, {}};
    for (int l = 0; l < L; ++l) {
      ring.lo.push_back(rs.lower(l));
      ring.di.push_back(rs.diag(l));
      ring.up.push_back(rs.upper(l));
    }
    std::vector<double> inv;
    if (!invert_dense(ring, inv)) return w.M = 0, false;
    const int rows = w.uniform ? 1 : L;
    for (int l = 0; l < rows; ++l) {
      std::vector<Blk> row(2 * D + 1);
      for (int d = -D; d <= D; ++d) {
        if (2 * D >= L && d == -D && L % 2 == 0) continue;  // lane l - L/2 is lane l + L/2
        if (d < -((L - 1) / 2) || d > L / 2) continue;
        std::copy_n(inv.begin() + ((size_t)l * L + rs.wrap(l + d)) * RR, RR, row[D + d].v);
      }
      put(row, D);
      w.gidx[l] = l;
    }
    return true;
  }
  // Lanes share a row when the sizes of the lanes in their window lie alike
  // (the inverse of the reduced system is the inverse of A at the interface
  // rows, in a cyclic line a function of the distance between them alone); in
  // an acyclic line also those beyond it, up to where its ends are felt
  std::map<std::vector<int>, int> seen;
  for (int l = 0; l < L; ++l) {
    if (w.uniform && l > 0) break;
    std::vector<int> key;
    const int reach = cyclic ? D : K + 1;
    for (int d = -reach; d < reach; ++d) {
      const int j = l + d;
      key.push_back(!cyclic && (j < 0 || j >= L) ? 2 : rs.type(rs.wrap(j)));
    }
    auto it = seen.find(key);
    if (it != seen.end()) {
      w.gidx[l] = it->second;
      continue;
    }
    if (!inverse_row(rs, l, K, g)) return w.M = 0, false;
    // (rows near the ends of an acyclic line, or between lanes of two sizes)
    double sum = 0.0, out = 0.0;
    for (int d = -K; d <= K; ++d) (std::abs(d) > D ? out : sum) += abs_sum(g[K + d], R);
    if (!(out <= tol * (sum + out))) return w.M = 0, false;
    const int at = (int)seen.size();
    seen[key] = at;
    w.gidx[l] = at;
    put(g, K);
  }
  return true;
}

bool build_window_rows(int n, int R, const double *bands, bool cyclic, int M, double tol, WinLayout &w) {
  using namespace window;
  const int W = 2 * R + 1, RR = R * R, RW = win_row_size(R);
  const int L = (n + M - 1) / M;
  if (L < 2 || L > 64 || (n + L - 1) / L != M || n / L < 2 * R + 1) return false;
  w = WinLayout();
  const int base = n / L, extra = n % L;
  auto a = [&](int g, int o) { return o < -R || o > R ? 0.0 : bands[(size_t)g * W + o + R]; };
  auto start = [&](int l) { return l * base + std::min(l, extra); };
  auto wrap = [&](int l) { return l < 0 ? l + L : (l >= L ? l - L : l); };
  auto rows_of = [&](int l) { return base + (l < extra ? 1 : 0) - R; };  // interior
  std::vector<double> top(n, 0.0);  // largest entry of each row: what is small or large is so beside it
  for (int j = 0; j < n; ++j)
    for (int o = -R; o <= R; ++o) top[j] = std::max(top[j], std::fabs(a(j, o)));
  std::vector<Blk> Sf(L), Sl(L), Rf(L), Rl(L), Lt(L), Dt(L), Ut(L);
  w.coef.assign((size_t)L * win_lane_size(R, M), 0.0);
  for (int l = 0; l < L; ++l) {
    const int i0 = start(l), m = rows_of(l), g0 = i0 + R;
    for (int i = 0; i < R; ++i)
      for (int c = 0; c < R; ++c) {
        Lt[l].v[i * R + c] = a(i0 + i, c - R - i);
        Dt[l].v[i * R + c] = a(i0 + i, c - i);
        Ut[l].v[i * R + c] = a(i0 + i, R + c - i);
      }
    // elimination of the interior; columns from m on are the next lane's
    std::vector<double> c((size_t)m * W), k((size_t)m * R, 0.0), u((size_t)m * R, 0.0), dinv(m);
    for (int j = 0; j < m; ++j)
      for (int o = -R; o <= R; ++o) c[(size_t)j * W + o + R] = j + o < 0 ? 0.0 : a(g0 + j, o);
    for (int j = 0; j < m; ++j) {
      const double piv = c[(size_t)j * W + R];
      if (!(std::fabs(piv) > 1e-2 * top[g0 + j]) || !std::isfinite(piv)) return false;
      dinv[j] = 1.0 / piv;
      for (int i = j + 1; i <= std::min(m - 1, j + R); ++i) {
        const double f = c[(size_t)i * W + (j - i + R)] / piv;
        k[(size_t)i * R + (i - j) - 1] = f;
        for (int q = j + 1; q <= j + R; ++q) c[(size_t)i * W + (q - i + R)] -= f * c[(size_t)j * W + (q - j + R)];
      }
      for (int q = 1; q <= R; ++q) u[(size_t)j * R + q - 1] = c[(size_t)j * W + R + q] * dinv[j];
    }
    auto forward = [&](double *x) {
      for (int j = 1; j < m; ++j)
        for (int q = 1; q <= R && q <= j; ++q) x[j] -= k[(size_t)j * R + q - 1] * x[j - q];
    };
    auto backward = [&](double *x) {
      for (int j = m - 1; j >= 0; --j) {
        double s = x[j] * dinv[j];
        for (int q = 1; q <= R && j + q < m; ++q) s -= u[(size_t)j * R + q - 1] * x[j + q];
        x[j] = s;
      }
    };
    double *row = w.coef.data() + (size_t)l * win_lane_size(R, M);
    std::vector<double> wf((size_t)R * m, 0.0), x(m);  // first R rows of U^{-1}
    for (int i = 0; i < R; ++i) {
      std::vector<double> p(m + R, 0.0);
      p[i] = 1.0;
      for (int j = i; j < m; ++j) {
        wf[(size_t)i * m + j] = p[j] * dinv[j];
        for (int q = 1; q <= R; ++q) p[j + q] -= p[j] * u[(size_t)j * R + q - 1];
      }
    }
    for (int s = 0; s < R; ++s) {
      for (int j = 0; j < m; ++j) x[j] = a(g0 + j, s - R - j);
      forward(x.data());
      for (int j = 0; j < m; ++j) row[(size_t)j * RW + 2 * R + s] = x[j];
      backward(x.data());
      for (int i = 0; i < R; ++i) {
        Sf[l].v[i * R + s] = x[i];
        Sl[l].v[i * R + s] = x[m - R + i];
      }
      for (int j = 0; j < m; ++j) x[j] = a(g0 + j, m + s - j);
      forward(x.data());
      backward(x.data());
      for (int i = 0; i < R; ++i) {
        Rf[l].v[i * R + s] = x[i];
        Rl[l].v[i * R + s] = x[m - R + i];
      }
    }
    bool bounded = true;  // the factors of the lane's rows, each of these divided by its largest entry
    auto note = [&](double v, double by) { bounded = bounded && std::fabs(v) <= 64.0 * by; };
    for (int j = 0; j < m; ++j) {
      double *t = row + (size_t)j * RW;
      for (int q = 0; q < R; ++q) {
        t[q] = k[(size_t)j * R + q];
        t[3 * R + 1 + q] = u[(size_t)j * R + q];
        for (int i = 0; i < R; ++i) t[R + q] += Ut[l].v[q * R + i] * wf[(size_t)i * m + j];
      }
      t[3 * R] = dinv[j];
      for (int q = 0; q < R; ++q) {
        if (q < j) note(t[q], top[g0 + j] / top[g0 + j - q - 1]);
        note(t[R + q], top[i0 + q] / top[g0 + j]);
        note(t[2 * R + q], top[g0 + j]);
        note(t[3 * R + 1 + q], 1.0);
      }
    }
    if (!bounded) return false;  // elimination that grows needs pivoting
    // z: the next lane's L~ times the last R rows of U^{-1}, on the last R values of z
    const int nx = wrap(l + 1), ni = start(nx);
    for (int i = 0; i < R; ++i) {
      std::fill(x.begin(), x.end(), 0.0);
      x[m - R + i] = 1.0;
      backward(x.data());
      for (int b = 0; b < R; ++b)
        for (int s = 0; s < R; ++s) row[(size_t)(M - R) * RW + b * R + i] += a(ni + b, s - R - b) * x[m - R + s];
    }
  }
  // the reduced system (Eqs. (18)-(20)) and its inverse; its rows are brought to
  // one size by powers of two, which the pivot search in a block needs
  double scale = 0.0;
  BlockRing ring{L, R, cyclic, std::vector<Blk>(L), std::vector<Blk>(L), std::vector<Blk>(L)};
  std::vector<Blk> &lo = ring.lo, &di = ring.di, &up = ring.up;
  std::vector<double> unit(L * R), inv;
  for (int l = 0; l < L; ++l) {
    di[l] = sub(Dt[l], mul(Ut[l], Sf[l], R), R);
    if (cyclic || l > 0) {
      di[l] = sub(di[l], mul(Lt[l], Rl[wrap(l - 1)], R), R);
      lo[l] = neg(mul(Lt[l], Sl[wrap(l - 1)], R), R);
    }
    if (cyclic || l < L - 1) up[l] = neg(mul(Ut[l], Rf[l], R), R);
    for (int i = 0; i < R; ++i) {
      double big = 0.0;
      for (const Blk *b : {&lo[l], &di[l], &up[l]})
        for (int c = 0; c < R; ++c) big = std::max(big, std::fabs(b->v[i * R + c]));
      const double u = big > 0.0 && std::isfinite(big) ? std::ldexp(1.0, -std::ilogb(big)) : 1.0;
      unit[l * R + i] = u;
      for (Blk *b : {&lo[l], &di[l], &up[l]})
        for (int c = 0; c < R; ++c) b->v[i * R + c] *= u;
    }
  }
  for (int i = 0; i < n * W; ++i) scale = std::max(scale, std::fabs(bands[i]));
  const bool done = R == 1 ? invert_blocks<1>(ring, inv) : (R == 2 ? invert_blocks<2>(ring, inv) : invert_blocks<3>(ring, inv));
  if (!done && !invert_dense(ring, inv)) return false;
  for (int l = 0; l < L; ++l)
    for (int j = 0; j < L; ++j)
      for (int i = 0; i < RR; ++i) inv[((size_t)l * L + j) * RR + i] *= unit[j * R + i % R];
  // the narrowest window that leaves out no more than tol of any lane's row
  auto dist = [&](int l, int j) {
    int d = j - l;
    if (cyclic && d > L / 2) d -= L;
    if (cyclic && d < -((L - 1) / 2)) d += L;
    return d;
  };
  int D = 1;
  for (int l = 0; l < L; ++l) {
    std::vector<double> far(L + 1, 0.0);
    double sum = 0.0, weight = 0.0;
    for (int j = 0; j < L; ++j)
      for (int i = 0; i < R; ++i)
        for (int c = 0; c < R; ++c) {
          const double v = std::fabs(inv[((size_t)l * L + j) * RR + i * R + c]);
          far[std::abs(dist(l, j))] += v * top[start(j) + c];
          weight += v * top[start(j) + c];
          sum += v;
        }
    if (!std::isfinite(sum) || !(sum * scale <= 1e4)) return false;
    double out = 0.0;
    int d = L;
    while (d > 0 && out + far[d] <= tol * weight) out += far[d--];
    D = std::max(D, d);
  }
  if (D > kWinMaxD || D > L - 1) return false;
  w.M = M;
  w.L = L;
  w.base = base;
  w.extra = extra;
  w.D = D;
  w.rows = 1;
  w.gidx.resize(L);
  w.g.assign((size_t)L * (2 * D + 1) * RR, 0.0);
  for (int l = 0; l < L; ++l) {
    w.gidx[l] = l;
    for (int j = 0; j < L; ++j) {
      const int d = dist(l, j);
      if (std::abs(d) > D) continue;
      std::copy_n(inv.begin() + ((size_t)l * L + j) * RR, RR, w.g.begin() + ((size_t)l * (2 * D + 1) + D + d) * RR);
    }
  }
  return true;
}

}  // namespace cb
