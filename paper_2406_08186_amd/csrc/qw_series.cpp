// Several CTQW time steps as one Chebyshev series.
//
// m steps of the order-K Taylor propagator are f(H) with
// f(x) = T_K(-i dt x)^m, a polynomial of degree K m.  On [-R, R], R a bound of
// ||H||, its Chebyshev coefficients fall below FP64 rounding after about
// m rho + 10 (m rho)^(1/3) terms (rho = dt R; Jacobi-Anger for a converged
// T_K), so f(H) psi needs that many products with H instead of K m: rho = 0.1,
// K = 20: 17 for 16 steps instead of 320; rho = 1, K = 13: 46 instead of 208.
// It is the same polynomial, evaluated in another basis, whatever K is: a
// short Taylor order keeps its own truncation error.
//
// f(-x) = conj f(x) on the real axis, so the coefficients are (-i)^k a_k with
// a_k real, and Clenshaw's recurrence for b_k = (-i)^k d_k has the form of a
// Horner stage:
//     d_k = a_k psi + d_{k+2} - 2i (H/R) d_{k+1},   k = M-1 .. 1,
//     f(H) psi = a_0 psi + d_2 - i (H/R) d_1,       d_M = a_M psi.
// A rounding error made in d_k reaches the result through T_k(H/R), whose norm
// is at most 1, so errors add without growth.

#include <cmath>
#include <complex>

#include "qw_plan.h"

namespace qwk {
namespace {

constexpr int kNodes = 192;           // Chebyshev nodes; coefficients alias only from degree 2 * 192 - 64 on
constexpr int kHalf = kNodes / 2;     // f at -x is conj f(x): half of them carry all values
constexpr int kProbe = 112;           // the coefficients up to here show that the series has ended
constexpr long double kDrop = 1e-17L; // a term this small changes no FP64 bit of a unit-norm state

struct Cosines {
  long double c[4 * kNodes];  // cos(pi j / (2 kNodes))
  Cosines() {
    const long double pi = 3.14159265358979323846264338327950288L;
    for (int j = 0; j < 4 * kNodes; ++j) c[j] = std::cos(pi * j / (2 * kNodes));
  }
};

}  // namespace

bool chebyshev_series(double rho, int K, int64_t steps, Series *out) {
  out->terms = 0;
  if (!(rho > 0.0) || steps < 1 || steps > kSeriesMaxSteps || rho * static_cast<double>(steps) > kSeriesMaxTerms)
    return false;
  static const Cosines table;
  long double re[kHalf], im[kHalf];
  for (int j = 0; j < kHalf; ++j) {
    // T_K(-i y), y = rho x_j, by Horner: p <- 1 + (-i y / k) p
    const long double y = rho * table.c[2 * j + 1];
    long double pr = 1.0L, pi = 0.0L;
    for (int k = K; k >= 1; --k) {
      const long double s = y / k, qr = 1.0L + s * pi, qi = -s * pr;
      pr = qr;
      pi = qi;
    }
    long double fr = 1.0L, fi = 0.0L;  // its power `steps`
    for (int64_t e = steps; e > 0; e >>= 1) {
      if (e & 1) {
        const long double t = fr * pr - fi * pi;
        fi = fr * pi + fi * pr;
        fr = t;
      }
      const long double t = pr * pr - pi * pi;
      pi = 2.0L * pr * pi;
      pr = t;
    }
    // a propagator far from unitary (Taylor order too short for its step) is left to the stages as written
    if (!(fr * fr + fi * fi < 4.0L)) return false;
    re[j] = fr;
    im[j] = fi;
  }
  long double tail = 0.0L;
  int last = -1;
  double a[kProbe + 1];
  for (int k = kProbe; k >= 0; --k) {
    long double s = 0.0L;
    const long double *v = (k & 1) ? im : re;  // even k: Re f, odd k: Im f
    for (int j = 0; j < kHalf; ++j) s += v[j] * table.c[(k * (2 * j + 1)) % (4 * kNodes)];
    s *= (k ? 4.0L : 2.0L) / kNodes;           // both halves of the nodes
    a[k] = static_cast<double>((k % 4 == 1 || k % 4 == 2) ? -s : s);
    if (last < 0) {
      tail += std::fabs(s);
      if (tail > kDrop) last = k;
    }
  }
  if (last < 2 || last > kSeriesMaxTerms) return false;
  out->terms = last;
  out->steps = steps;
  for (int k = 0; k <= kSeriesMaxTerms + 1; ++k) out->a[k] = k <= last ? a[k] : 0.0;
  return true;
}

}  // namespace qwk
