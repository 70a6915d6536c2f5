// The sign-change count of the resident spectral norm (minors.inc, taken
// from spectral_run.hip) on the CPU: small tridiagonals and points with exact
// minors, many of them eigenvalues, where the last minor is zero and only
// padding rows follow; the count is that of the rows alone. Random ones of
// every order against the count of the LDL^T pivots. Prints "ok".
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <random>

#define __device__
#define __forceinline__ inline

namespace {

typedef double f64x2 __attribute__((vector_size(16)));
using std::isfinite;

#include "minors.inc"

struct Scaled {
  alignas(16) double a[64], b2[64];
};

// Sign changes of the leading minors of the m rows; a zero one has the sign
// opposite to the one before it.
int reference(const Scaled& t, int m, double x) {
  double p0 = 0.0, p1 = 1.0;
  bool neg = false;
  int cnt = 0;
  for (int i = 0; i < m; ++i) {
    const double p2 = (t.a[i] - x) * p1 - t.b2[i] * p0;
    const bool ng = (p2 == 0.0) ? !neg : p2 < 0.0;
    cnt += ng != neg;
    neg = ng;
    p0 = p1;
    p1 = p2;
  }
  return cnt;
}

int pivots(const Scaled& t, int m, double x) {
  int cnt = 0;
  double d = 1.0;
  for (int i = 0; i < m; ++i) {
    d = t.a[i] - x - (i > 0 ? t.b2[i] / d : 0.0);
    if (d == 0.0) d = -1e-300;
    cnt += d < 0.0;
  }
  return cnt;
}

}  // namespace

int main() {
  std::mt19937 g(5);
  int bad = 0, zeros = 0;
  auto fail = [&](const char* what, int m, double x, int got, int want) {
    if (bad++ < 10) fprintf(stderr, "%s: order %d at %g: %d, not %d\n", what, m, x, got, want);
  };
  Scaled t;
  // eigenvalues 0 and 1
  for (int i = 0; i < 64; ++i)
    t.a[i] = i < 2 ? 0.5 : 2.0, t.b2[i] = i == 1 ? 0.25 : (i == 2 ? kPadLink : 0.0);
  for (double x : {0.0, 1.0})
    if (minors_below(t.a, t.b2, 1, x) != (x == 0.0 ? 1 : 2))
      fail("2 x 2", 2, x, minors_below(t.a, t.b2, 1, x), x == 0.0 ? 1 : 2);
  for (int it = 0; it < 400000; ++it) {
    const int m = 1 + g() % 8;
    for (int i = 0; i < 64; ++i) {
      t.a[i] = i < m ? (static_cast<int>(g() % 9) - 4) / 8.0 : 2.0;
      const double b = (i > 0 && i < m) ? (1 + g() % 2) / 4.0 : 0.0;
      t.b2[i] = (i == m) ? kPadLink : b * b;
    }
    const double x = (static_cast<int>(g() % 17) - 8) / 8.0;
    const int got = minors_below(t.a, t.b2, (m + 7) / 8, x), want = reference(t, m, x);
    double p0 = 0.0, p1 = 1.0;
    for (int i = 0; i < m; ++i) {
      const double p2 = (t.a[i] - x) * p1 - t.b2[i] * p0;
      p0 = p1;
      p1 = p2;
    }
    zeros += p1 == 0.0;
    if (got != want) fail("exact", m, x, got, want);
  }
  std::uniform_real_distribution<double> u(0.0, 1.0);
  for (int it = 0; it < 100000; ++it) {
    const int m = 1 + g() % 64;
    for (int i = 0; i < 64; ++i) {
      t.a[i] = i < m ? u(g) - 0.5 : 2.0;
      const double b = (i > 0 && i < m) ? 0.25 * u(g) * (g() % 9 ? 1.0 : 1e-12) : 0.0;
      t.b2[i] = (i == m) ? kPadLink : b * b;
    }
    const double x = 2.0 * u(g) - 1.0;
    if (minors_below(t.a, t.b2, (m + 7) / 8, x) != pivots(t, m, x))
      fail("random", m, x, minors_below(t.a, t.b2, (m + 7) / 8, x), pivots(t, m, x));
  }
  if (zeros < 1000) ++bad;
  if (!bad) printf("ok\n");
  return bad != 0;
}
