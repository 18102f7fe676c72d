// The parts of the hierarchical summation that run on the host: the layout of a square's record, the order of the
// coefficients, the Hilbert index, and the expansion with its order rule against direct float64 sums.
#include <math.h>
#include <stdio.h>

#include <complex>
#include <set>
#include <vector>

#include "tree_core.h"

using namespace aidw::tree;

static int failures = 0;
#define CHECK(cond, ...)                        \
  do {                                          \
    if (!(cond)) {                              \
      ++failures;                               \
      printf("%s:%d: ", __FILE__, __LINE__);    \
      printf(__VA_ARGS__);                      \
      printf("\n");                             \
    }                                           \
  } while (0)

static double uniform(uint64_t& state) {
  state = state * 6364136223846793005ull + 1442695040888963407ull;
  return (double)(state >> 11) * 0x1p-53;
}

static void layout() {
  std::set<int> used;
  int at = 0;
  for (int o = 0; o <= kOrder; ++o)
    for (int l = o & 1; l <= o; l += 2) {
      const int m = (o - l) / 2, off = coef_offset(l, m), len = l == 0 ? 2 : 4;
      CHECK(coef_place(l + m, m) == at++, "place of (%d, %d)", l, m);
      CHECK(off >= 4 && off + len <= kChild && off % len == 0, "offset of (%d, %d) is %d", l, m, off);
      for (int i = 0; i < len; ++i) CHECK(used.insert(off + i).second, "(%d, %d) overlaps another", l, m);
    }
  CHECK(at == kCoefs, "%d coefficients", at);
  for (int bits = 1; bits <= 6; ++bits) {  // every tile once, neighbours along the curve side by side
    std::vector<int> x(1 << (2 * bits), -1), y(x);
    for (int i = 0; i < 1 << bits; ++i)
      for (int j = 0; j < 1 << bits; ++j) {
        const uint32_t d = hilbert(bits, i, j);
        CHECK(d < x.size() && x[d] < 0, "tile (%d, %d) of %d bits", i, j, bits);
        x[d] = i;
        y[d] = j;
      }
    for (size_t d = 1; d < x.size(); ++d)
      CHECK(abs(x[d] - x[d - 1]) + abs(y[d] - y[d - 1]) == 1, "step %zu of %d bits", d, bits);
  }
}

// A square's record (double), its points about the centre 0 with side 1.
static void expansion(double alpha, uint64_t seed) {
  uint64_t state = seed;
  const int n = 40;
  std::vector<std::complex<double>> r(n);
  std::vector<double> z(n);
  for (int i = 0; i < n; ++i) {
    r[i] = {uniform(state) - 0.5, uniform(state) - 0.5};
    if (i < 4) r[i] = {i & 1 ? 0.5 : -0.5, i & 2 ? 0.5 : -0.5};
    z[i] = uniform(state) - 0.3;
  }
  double rec[kRec] = {}, sabs = 0.0;
  for (int i = 0; i < n; ++i) {
    sabs += fabs(z[i]);
    for (int l = 0; l <= kOrder; ++l)
      for (int m = 0; l + 2 * m <= kOrder; ++m) {
        const std::complex<double> p = std::pow(r[i], l) * std::pow(std::norm(r[i]), m) * (l ? 2.0 : 1.0);
        double* c = rec + coef_offset(l, m);
        c[0] += z[i] * p.real();
        c[l ? 2 : 1] += p.real();
        if (l) {
          c[1] += z[i] * p.imag();
          c[3] += p.imag();
        }
      }
  }
  double b[kOrder + 1] = {1.0};
  for (int j = 1; j <= kOrder; ++j) b[j] = b[j - 1] * (0.5 * alpha + j - 1) / j;
  for (int tier = 0; tier < kTiers; ++tier) {
    const int P = 2 * tier + 2;
    // the nearest place at which the rule takes this order, for a square that makes up the whole sums
    const double rho = fmin(exp2(order_bound(alpha, tier) / (P + 1)), 0.4714);
    for (int a = 0; a < 8; ++a) {
      const std::complex<double> q = std::polar(M_SQRT1_2 / rho, 0.3 + a * M_PI / 4);
      const std::complex<double> v = q / std::norm(q);
      double num = 0.0, den = 0.0, wz = 0.0, w = 0.0;
      for (int l = 0; l <= P; ++l)
        for (int m = 0; l + 2 * m <= P; ++m) {
          const double* c = rec + coef_offset(l, m);
          const std::complex<double> f = std::conj(std::pow(v, l)) * std::pow(std::norm(v), m) * b[l + m] * b[m];
          num += l ? (std::complex<double>(c[0], c[1]) * f).real() : c[0] * f.real();
          den += l ? (std::complex<double>(c[2], c[3]) * f).real() : c[1] * f.real();
        }
      for (int i = 0; i < n; ++i) {
        const double wi = pow(std::abs(q - r[i]) / std::abs(q), -alpha);
        wz += wi * z[i];
        w += wi;
      }
      CHECK(fabs(num - wz) <= 3 * 0x1p-22 * sabs && fabs(den - w) <= 3 * 0x1p-22 * n,
            "alpha %g order %d: num off by %.2e, den by %.2e", alpha, P, fabs(num - wz) / sabs, fabs(den - w) / n);
    }
  }
}

int main() {
  layout();
  const double alphas[] = {0.05, 0.5, 1, 2, 3.25, 5, 8};
  for (int i = 0; i < 7; ++i)
    for (uint64_t s = 0; s < 4; ++s) expansion(alphas[i], 17 * s + i);
  printf("%d failures\n", failures);
  return failures != 0;
}
