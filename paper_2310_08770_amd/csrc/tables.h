// Tables of the correlation passes and of the window expansion (refine.hip),
// built on the host in FP64.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <vector>

#include "common.h"

namespace ccpt {

// Half width B (px) of the window expansion: it covers every grid offset and
// every displacement the window test accepts, with a little room for Newton
// iterates on the way.
inline double window_half(double half_window, int u, int M, int c) {
  const double grid = (double)(c > M - 1 - c ? c : M - 1 - c) / u;
  return (grid > half_window ? grid : half_window) + 0.05;
}

// J_n(z), n < count, by downward recurrence normalised with
// J_0 + 2 (J_2 + J_4 + ...) = 1 (Miller's algorithm; z below 4 here).
inline void bessel_j(double z, int count, double* j) {
  if (z == 0.0) {
    for (int n = 0; n < count; ++n) j[n] = n ? 0.0 : 1.0;
    return;
  }
  const int top = 80;
  double hi = 0.0, cur = 1e-280, sum = 0.0;
  for (int n = top; n >= 0; --n) {  // cur = J_n, hi = J_{n+1} (unnormalised)
    if (n < count) j[n] = cur;
    if (n % 2 == 0) sum += n ? 2.0 * cur : cur;
    const double lo = n ? 2.0 * n / z * cur - hi : 0.0;
    hi = cur;
    cur = lo;
    if (std::fabs(cur) > 1e200) {
      cur *= 1e-200;
      hi *= 1e-200;
      sum *= 1e-200;
      for (int k = n; k < count; ++k) j[k] *= 1e-200;
    }
  }
  for (int n = 0; n < count; ++n) j[n] /= sum;
}

// Weights g[n] (n < kChebN) of the series of exp(i z x): cos(z x) =
// sum over even n of g[n] T_n(x), sin(z x) = sum over odd n.
inline void cheb_weights(double z, double* g) {
  double j[kChebN];
  bessel_j(z, kChebN, j);
  for (int n = 0; n < kChebN; ++n) g[n] = ((n / 2) & 1 ? -1.0 : 1.0) * (n ? 2.0 : 1.0) * j[n];
}

// Twiddles exp(-2 pi i m / n), m < n.
inline std::vector<double2> twiddles(int n) {
  std::vector<double2> t(n);
  for (int m = 0; m < n; ++m) {
    const double a = 2.0 * M_PI * (double)m / (double)n;
    t[m] = make_double2(std::cos(a), -std::sin(a));
  }
  return t;
}

struct ShapeTables {
  std::vector<double2> gy, gx;
  std::vector<double> gxn;
  int ksteps = 0;
};

// Tables of frames of ny rows of nx pixels for the half width `half`.
inline ShapeTables build_shape_tables(int ny, int nx, double half) {
  ShapeTables t;
  const int nq = ny / 2, nc = nx / 2, tiles = window_tiles(nx);
  t.ksteps = (nq + 1 + 3) / 4;
  t.gy.assign((size_t)t.ksteps * 64, make_double2(0.0, 0.0));
  double g[kChebN];
  for (int q = 0; q <= nq; ++q) {
    cheb_weights(2.0 * M_PI * q * half / ny, g);
    const double w = (q == 0 || q == nq) ? 0.5 : 1.0;  // these rows pair with themselves
    for (int i = 0; i < kChebN / 2; ++i)
      t.gy[(size_t)(q / 4) * 64 + (q % 4) * 16 + i] = make_double2(w * g[2 * i], w * g[2 * i + 1]);
  }
  // column kx = 16 tile + 4 v + lane / 16 of k step (tile, v); m = 2 (lane mod
  // 16) and that + 1.  Re[(..) i^m] takes Re for even m and -Im for odd m.
  t.gx.assign((size_t)tiles * 4 * 64, make_double2(0.0, 0.0));
  const double inv = 1.0 / ((double)ny * (double)nx);
  for (int kx = 0; kx < nc; ++kx) {
    cheb_weights(2.0 * M_PI * kx * half / nx, g);
    const double w = (kx ? 2.0 : 1.0) * inv;
    for (int i = 0; i < kChebN / 2; ++i)
      t.gx[((size_t)(kx / 16) * 4 + kx % 16 / 4) * 64 + (kx % 4) * 16 + i] =
          make_double2(w * g[2 * i], -w * g[2 * i + 1]);
  }
  cheb_weights(M_PI * half, g);
  for (int i = 0; i < kChebN / 2; ++i) t.gxn.push_back(inv * g[2 * i]);
  return t;
}

struct GridTables {
  std::vector<float> tf;
  std::vector<double> td;
};

// T_n at the grid offsets (m - c)/u, in units of `half`.
inline GridTables build_grid_tables(int u, int M, int c, double half) {
  GridTables t;
  const int m32 = (M + 31) / 32 * 32, m16 = (M + 15) / 16 * 16;
  t.tf.assign((size_t)m32 * kGridN, 0.f);
  t.td.assign((size_t)m16 * kChebN, 0.0);
  for (int m = 0; m < M; ++m) {
    const double x = (double)(m - c) / u / half;
    double a = 1.0, b = x;  // T_n, T_{n+1}
    for (int n = 0; n < kChebN; ++n) {
      if (n < kGridN) t.tf[(size_t)m * kGridN + n] = (float)a;
      t.td[(size_t)m * kChebN + n] = a;
      const double next = 2.0 * x * b - a;
      a = b;
      b = next;
    }
  }
  return t;
}

}  // namespace ccpt
