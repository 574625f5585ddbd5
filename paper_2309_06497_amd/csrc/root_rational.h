// Rational approximation of x^-r, 0 < r < 1, for the root inverses that do without eigenvectors
// (root_tridiag.h, root_band.h).
//
//     x^-r  ~=  sum_j w_j / (x + s_j)      for lo <= x <= hi
//
// turns f(A) = (A - min(lambda_min, 0) I + eps I)^-r into a sum of inverses of shifted matrices.
// For a tridiagonal or banded matrix every one of those is a few recurrences, and nothing in it
// needs eigenvectors to be computed, told apart or kept orthogonal.
//
// The poles are spaced evenly on a logarithmic axis, from e^-3 lo to e^4 hi; the weights are the
// least-squares fit of the relative error over [lo, hi] (the Stieltjes integral of x^-r by the
// trapezoidal rule on that axis, with its two infinite tails folded into the outermost weights).
// With 7 + 0.866 ln(hi / lo) poles the relative error is below 1.3e-7 at r = 1/4 and 2.3e-7 at r = 1/2.
// rat_table accepts 4e-7, which is r <= 0.663 (2/3 would be 4.1e-7); above, the poles would have to reach further down.
// hi / lo comes in classes of 2^4, 2^8, ... 2^48, so that a matrix pays for the spread that it has.
#pragma once
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

namespace shampoo {

constexpr int RAT_CLASSES = 12;          // class c: hi / lo = 2^(4 (c + 1))
constexpr int RAT_MAX_POLES = 36;
constexpr int RAT_WEIGHTS = 276;         // of all classes together
constexpr double RAT_BELOW = 3.0, RAT_ABOVE = 4.0;   // how far the poles reach beyond [ln lo, ln hi]

__host__ __device__ constexpr int rat_poles(int c) { return 7 + (240 * (c + 1) + 99) / 100; }   // 7 + ceil(0.866 ln 2^(4 (c + 1)))
__host__ __device__ constexpr int rat_offset(int c) { int o = 0; for (int k = 0; k < c; ++k) o += rat_poles(k); return o; }
static_assert(rat_poles(RAT_CLASSES - 1) == RAT_MAX_POLES && rat_offset(RAT_CLASSES) == RAT_WEIGHTS, "pole counts");

// Weights for lo = 1; travels as a kernel argument.  x^-r = lo^(1 - r) sum_j w[j] / (x + lo s_j).
struct RatTable { double w[RAT_WEIGHTS]; };

// ln of pole j of class c, for lo = 1
__host__ __device__ inline double rat_log_pole(int c, int j) {
  const double span = 4.0 * (c + 1) * 0.6931471805599453;
  return -RAT_BELOW + j * ((span + RAT_BELOW + RAT_ABOVE) / (rat_poles(c) - 1));
}
// smallest class whose range holds hi / lo
__host__ __device__ inline int rat_class(double lo, double hi) {
  int c = 0;
  while (c < RAT_CLASSES - 1 && hi > ldexp(lo, 4 * (c + 1))) ++c;
  return c;
}

// Least squares by Householder QR, columns scaled to 1; false if the fit is not good enough.
inline bool rat_fit(double r, RatTable &t) {
  if (!(r > 0.0 && r < 1.0)) return false;
  for (int c = 0; c < RAT_CLASSES; ++c) {
    const int np = rat_poles(c), m = 6 * np + 1;
    const double span = 4.0 * (c + 1) * 0.6931471805599453;
    std::vector<double> s(np), a((size_t)m * (np + 1)), sc(np);
    for (int j = 0; j < np; ++j) s[j] = std::exp(rat_log_pole(c, j));
    for (int i = 0; i < m; ++i) {      // points denser towards both ends of the range
      const double x = std::exp(span * 0.5 * (1.0 - std::cos(3.14159265358979324 * i / (m - 1)))), xr = std::pow(x, r);
      for (int j = 0; j < np; ++j) a[(size_t)j * m + i] = xr / (x + s[j]);
      a[(size_t)np * m + i] = 1.0;
    }
    for (int j = 0; j < np; ++j) {
      double big = 0.0;
      for (int i = 0; i < m; ++i) big = std::max(big, a[(size_t)j * m + i]);
      sc[j] = big;
      for (int i = 0; i < m; ++i) a[(size_t)j * m + i] /= big;
    }
    for (int j = 0; j < np; ++j) {     // column j: reflector in place, applied to the columns right of it
      double *v = &a[(size_t)j * m];
      double nrm = 0.0;
      for (int i = j; i < m; ++i) nrm += v[i] * v[i];
      nrm = std::sqrt(nrm);
      const double alpha = v[j] > 0.0 ? -nrm : nrm, v0 = v[j] - alpha;
      const double vv = nrm * nrm - alpha * v[j] * 2.0 + alpha * alpha;   // |v - alpha e|^2
      if (!(vv > 0.0)) return false;
      v[j] = v0;
      for (int k = j + 1; k <= np; ++k) {
        double *u = &a[(size_t)k * m];
        double dot = 0.0;
        for (int i = j; i < m; ++i) dot += v[i] * u[i];
        dot *= 2.0 / vv;
        for (int i = j; i < m; ++i) u[i] -= dot * v[i];
      }
      v[j] = alpha;                    // R's diagonal; the rest of the reflector is not needed again
    }
    double *w = t.w + rat_offset(c);
    const double *y = &a[(size_t)np * m];
    for (int j = np - 1; j >= 0; --j) {
      double x = y[j];
      for (int k = j + 1; k < np; ++k) x -= a[(size_t)k * m + j] * w[k];
      w[j] = x / a[(size_t)j * m + j];
    }
    for (int j = 0; j < np; ++j) w[j] /= sc[j];
    for (int i = 0; i <= 10 * np; ++i) {
      const double x = std::exp(span * i / (10 * np));
      double f = 0.0;
      for (int j = 0; j < np; ++j) f += w[j] / (x + s[j]);
      if (!(std::fabs(f * std::pow(x, r) - 1.0) <= 4e-7)) return false;
    }
  }
  return true;
}

// The table of exponent r, or nullptr where the fit does not hold (r outside (0, 1) or close to its
// ends).  A program uses one exponent, or three where its tensors have different orders: the
// last few are kept.
inline bool rat_table(float r, RatTable &out) {
  struct Entry { float r; bool ok; RatTable t; };
  static std::mutex mutex;
  static Entry entries[8];
  static int used = 0, next = 0;
  std::lock_guard<std::mutex> lock(mutex);
  for (int i = 0; i < used; ++i)
    if (entries[i].r == r) {
      if (entries[i].ok) std::memcpy(&out, &entries[i].t, sizeof(out));
      return entries[i].ok;
    }
  Entry &e = entries[next];
  next = (next + 1) % 8;
  used = std::max(used, next == 0 ? 8 : next);
  e.r = r;
  e.ok = rat_fit((double)r, e.t);
  if (e.ok) std::memcpy(&out, &e.t, sizeof(out));
  return e.ok;
}

}  // namespace shampoo
