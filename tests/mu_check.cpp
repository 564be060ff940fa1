// Host check of the chemical-potential search of the library.
#include "gw_mu.h"
#include <cmath>
#include <cstdio>
#include <functional>
#include <limits>

static int bad = 0;
#define CHECK(c)                                                \
  do {                                                          \
    if (!(c)) { ++bad; printf("line %d: %s\n", __LINE__, #c); } \
  } while (0)

using Fn = std::function<double(double)>;

// matrices of more than 32 orbitals are inverted one mu after another, and a
// launch's partial sums stay within 2 MB (or one count)
static void batch_rule() {
  for (long long m : {2LL, 24LL, 273LL, 1000LL, 4096LL, 6400LL, 65536LL, 2048LL * 262144LL})
    for (int nao = 1; nao <= 60; ++nao) {
      const MuCounts c = mu_counts(nao, m);
      CHECK(c.batch >= 1 && c.ahead >= c.batch && c.ahead <= kMuBatch);
      CHECK(c.ahead == 1 || c.ahead * m <= 262144);
      if (nao > 32) CHECK(c.ahead == 1);
    }
  auto is = [](int nao, long long m, int batch, int ahead) {
    const MuCounts c = mu_counts(nao, m);
    return c.batch == batch && c.ahead == ahead;
  };
  CHECK(is(6, 192, 15, 15) && is(8, 1000, 7, 15) && is(12, 1200, 3, 15) && is(20, 1200, 1, 15) && is(26, 1200, 1, 1));
}

// the plain bisection, and how many counts it asks for
static gw_status plain(const Fn& f, double target, double tol, double mu0, double* out, int* counts) {
  double lo = mu0 - 1.0, hi = mu0 + 1.0, step = 1.0, n;
  *counts = 0;
  auto at = [&](double x) { ++*counts; n = f(x); return std::isfinite(n); };
  for (int it = 0;;) {
    if (!at(lo)) return std::isinf(n) ? GW_ERR_SINGULAR : GW_ERR_NONFINITE;
    if (!(n > target)) break;
    step *= 2.0;
    lo -= step;
    if (++it > 60) return GW_ERR_NOCONV;
  }
  step = 1.0;
  for (int it = 0;;) {
    if (!at(hi)) return std::isinf(n) ? GW_ERR_SINGULAR : GW_ERR_NONFINITE;
    if (!(n < target)) break;
    step *= 2.0;
    hi += step;
    if (++it > 60) return GW_ERR_NOCONV;
  }
  for (int it = 0; hi - lo > tol && it < 400; ++it) {
    const double mid = 0.5 * (lo + hi);
    if (!at(mid)) return std::isinf(n) ? GW_ERR_SINGULAR : GW_ERR_NONFINITE;
    (n < target ? lo : hi) = mid;
  }
  *out = 0.5 * (lo + hi);
  return hi - lo > tol ? GW_ERR_NOCONV : GW_OK;
}

struct Given {
  const Fn* f;
  int batch;
  int *launches, *counts;
  gw_status operator()(const double* mu, int n, double* ne) const {
    CHECK(n >= 1 && n <= batch);
    ++*launches;
    *counts += n;
    for (int i = 0; i < n; ++i) ne[i] = (*f)(mu[i]);
    return GW_OK;
  }
};

// the same status and bits as the plain bisection for every batch; most: launches of 15
static void same(const char* name, const Fn& f, double target, double tol, double mu0, int most) {
  double want = 0.0;
  int np = 0;
  const gw_status ws = plain(f, target, tol, mu0, &want, &np);
  for (int batch : {1, 2, 3, 4, 7, 8, 14, 15})
  for (int ahead : {batch, 15}) {
    int launches = 0, counts = 0;
    double got = 0.0;
    MuRoot<Given> r{Given{&f, std::max(batch, ahead), &launches, &counts}, batch, ahead, target, tol};
    const gw_status s = r.find(mu0, &got);
    CHECK(s == ws);
    CHECK(s == GW_OK ? got == want : *r.why != 0);
    CHECK(launches <= np);
    if (ahead == 1 && s == GW_OK) CHECK(launches == np && counts == np);
    if (batch == 15 && launches > most) {
      ++bad;
      printf("%s: %d launches\n", name, launches);
    }
    if (s == GW_OK && (batch == 1 || batch == 3 || batch == 15))
      printf("%-10s batch %2d ahead %2d: %3d launches, %3d counts\n", name, batch, ahead, launches, counts);
  }
}

static double fermi(double x) { return x > 0 ? 1.0 / (1.0 + std::exp(-x)) : std::exp(x) / (1.0 + std::exp(x)); }

int main() {
  batch_rule();
  const double tol = 1e-13;
  // levels e of an occupied and an empty band at beta, with an error of the size err of the count
  auto levels = [](double beta, double lo1, double hi1, double lo2, double hi2, double err) {
    return [=](double mu) {
      double n = 0.0;
      for (int i = 0; i < 64; ++i) {
        const double u = (i + 0.5) / 64;
        n += fermi(beta * (mu - lo1 - u * (hi1 - lo1))) / 32 + fermi(beta * (mu - lo2 - u * (hi2 - lo2))) / 32;
      }
      return n + err * std::sin(37.0 * mu + 1.0);
    };
  };
  for (double mu0 : {0.0, 0.31, -2.7}) {
    same("metal", levels(50.0, -1.0, 0.0, 0.0, 1.0, 0.0), 1.7, tol, mu0, 11);
    same("cold metal", levels(1000.0, -1.0, 0.0, 0.0, 1.0, 0.0), 1.7, tol, mu0, 13);
    // flat in the gap: rounding decides, and a count that falls with mu there
    same("gap", levels(200.0, -1.0, -0.5, 0.5, 1.0, 0.0), 2.0, tol, mu0, 14);
    same("ripple", levels(200.0, -1.0, -0.5, 0.5, 1.0, 1e-9), 2.0, tol, mu0, 14);
    same("rough", levels(200.0, -1.0, -0.5, 0.5, 1.0, 1e-2), 2.0, tol, mu0, 14);
    // several roots far from each other
    same("roots", [](double x) { return 1.0 + 0.5 * std::tanh(3.0 * x) + 0.9 * std::sin(9.0 * x); }, 1.1, tol, mu0, 14);
    same("step", [](double x) { return x < 0.123456789 ? 0.5 : 1.5; }, 1.0, tol, mu0, 14);
    same("line", [](double x) { return 1.0 + 0.1 * x; }, 1.01, tol, mu0, 14);
    same("coarse", levels(50.0, -1.0, 0.0, 0.0, 1.0, 0.0), 1.7, 1e-3, mu0, 6);
  }
  const double nan = std::numeric_limits<double>::quiet_NaN(), inf = std::numeric_limits<double>::infinity();
  // no bracket; a bracket that cannot be narrowed to tol
  same("full", [](double) { return 1.0; }, 1.5, tol, 0.0, 62);
  same("empty", [](double) { return 1.0; }, 0.5, tol, 0.0, 62);
  same("far", [](double x) { return x - 1e6; }, 0.25, tol, 1e6, 60);
  // counts that the bisection needs and that are not finite
  same("nan", [=](double x) { return std::fabs(x - 0.5) < 0.01 ? nan : x; }, 0.6, tol, 0.0, 14);
  same("pivot", [=](double x) { return x == 0.5 ? inf : x; }, 0.6, tol, 0.0, 14);
  // and that it does not need
  same("nan off", [=](double x) { return std::fabs(x + 0.5) < 0.01 ? nan : x; }, 0.6, tol, 0.0, 14);
  same("pivot off", [=](double x) { return x == -0.5 ? -inf : x; }, 0.6, tol, 0.0, 14);
  printf("bad %d\n", bad);
  return bad != 0;
}
