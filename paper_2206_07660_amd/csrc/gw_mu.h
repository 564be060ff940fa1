// Host side of the chemical-potential search (internal).
#pragma once
#include <algorithm>
#include <cmath>

#include "../../include/gw.h"

constexpr int kMuBatch = 15;   // most values of mu in one launch

// Values of mu whose electron counts one launch takes, for `matrices` = nw_f nk
// Dyson matrices of order nao.  The wave-per-matrix inversion (nao <= 32) takes
// several at once: up to 15 while their waves leave the chip's 8192 wave slots
// half empty, where one more value costs little more.  Larger matrices
// are inverted one value of mu after another, so a second value costs as much
// as the first: with 15 of them asked for, a search at nao 33 .. 60 (2x2x2, 24
// frequencies) took 9.7 .. 29 ms, the plain bisection 6.2 .. 15 ms.
inline int mu_batch(int nao, long long matrices) {
  if (nao > 32) return 1;
  return (int)std::max(1LL, std::min((long long)kMuBatch, 4096LL / matrices));
}

// Whether a count that is needed can be used: an infinite one marks a zero pivot.
inline gw_status count_status(double n, const char** why) {
  if (std::isfinite(n)) return GW_OK;
  *why = std::isinf(n) ? "electron count: zero pivot" : "electron count is not finite";
  return std::isinf(n) ? GW_ERR_SINGULAR : GW_ERR_NONFINITE;
}

// Root of N_e(mu) = target by bracket expansion from mu0 +- 1 Ha and bisection
// to a bracket of tol.  Every decision is a count at its own midpoint: N_e need
// not rise with mu (a gap at low temperature, where it is flat up to the error
// of the sparse grids, or a self-energy that is not causal), so that counts
// elsewhere say nothing about a midpoint, and where it has several roots the
// order of the midpoints picks one.  A launch takes `batch` counts: all
// midpoints of the next levels (four levels of 15 counts) or, once the secant
// of a bracket has fallen into the bracket that followed, the midpoints on the
// way to the secant's root, 15 levels if it is right (each such launch about
// doubles the known digits).  Counts that the plain bisection would not have
// asked for decide nothing.  One search to 1e-13 takes 47 launches of one
// count, 13 to 15 of four or 5 to 9 of 15 for a metal, 17 to 23 or 10 to 14 in
// a gap: 0.18 / 0.22 ms at 2x2x2, nao 6, 24 frequencies, 0.88 / 1.3 ms at 3x3x3,
// nao 16, 60, and 5.5 / 5.5 ms at 4x4x4, nao 26, 100 (metal / gap; 1.9, 3.8 and
// 16.9 ms with one workgroup-wide inversion and one copied count at a time).
// Taking counts to rise with mu, and skipping the midpoints that this settles,
// gives 0.20 / 0.34, 0.43 / 1.5 and 1.9 / 5.9 ms, but has moved mu by 0.2 Ha in
// a gap (beta 1000, 24 nodes).
//
// at(mu, n, ne) forms the counts ne[i] at mu[i], i < n <= batch.
template <class Count>
struct MuRoot {
  Count at;
  int batch;
  double target, tol;
  const char* why = "";   // of a status that is not GW_OK and not at()'s own

  gw_status find(double mu0, double* out) {
    double lo = mu0 - 1.0, hi = mu0 + 1.0, step = 1.0, nlo = 0.0, nhi = 0.0;
    gw_status s;
    if (batch >= 2) {
      const double mu[2] = {lo, hi};
      double ne[2];
      if ((s = at(mu, 2, ne)) != GW_OK) return s;
      nlo = ne[0];
      nhi = ne[1];
    } else if ((s = at(&lo, 1, &nlo)) != GW_OK) {
      return s;
    }
    if ((s = usable(nlo)) != GW_OK) return s;
    for (int it = 0; nlo > target;) {
      step *= 2.0;
      lo -= step;
      if (++it > 60) return no("mu search: no lower bracket");
      if ((s = one(lo, &nlo)) != GW_OK) return s;
    }
    if (batch < 2 && (s = at(&hi, 1, &nhi)) != GW_OK) return s;
    if ((s = usable(nhi)) != GW_OK) return s;
    step = 1.0;
    for (int it = 0; nhi < target;) {
      step *= 2.0;
      hi += step;
      if (++it > 60) return no("mu search: no upper bracket");
      if ((s = one(hi, &nhi)) != GW_OK) return s;
    }
    bool follow = false;                      // the secant's root is worth following
    for (int it = 0; hi - lo > tol && it < 400;) {
      const double x = lo + (hi - lo) * ((target - nlo) / (nhi - nlo));
      double mu[kMuBatch], ne[kMuBatch];
      const int n = follow ? way(lo, hi, x, mu) : tree(lo, hi, mu), it0 = it;
      if ((s = at(mu, n, ne)) != GW_OK) return s;
      while (hi - lo > tol && it < 400) {
        const double mid = 0.5 * (lo + hi);
        int i = 0;
        while (i < n && mu[i] != mid) ++i;
        if (i == n) break;
        if ((s = usable(ne[i])) != GW_OK) return s;
        if (ne[i] < target) {
          lo = mid;
          nlo = ne[i];
        } else {
          hi = mid;
          nhi = ne[i];
        }
        ++it;
      }
      // a way that brought less than the levels of a tree is not taken again
      follow = follow ? (2 << std::min(it - it0, 20)) > n + 1 : x > lo && x < hi;
    }
    if (hi - lo > tol) return no("mu search: bracket not narrowed to tol");
    *out = 0.5 * (lo + hi);
    return GW_OK;
  }

 private:
  gw_status no(const char* text) {
    why = text;
    return GW_ERR_NOCONV;
  }
  gw_status usable(double n) { return count_status(n, &why); }
  gw_status one(double mu, double* n) {
    const gw_status s = at(&mu, 1, n);
    return s == GW_OK ? usable(*n) : s;
  }
  // midpoints of the next levels of [lo, hi], level by level
  int tree(double lo, double hi, double* mu) const {
    struct { double lo, hi; } node[kMuBatch] = {{lo, hi}};
    int n = 0;
    for (int cnt = 1; n < cnt; ++n) {
      const double l = node[n].lo, h = node[n].hi;
      mu[n] = 0.5 * (l + h);
      if (cnt < batch) node[cnt++] = {l, mu[n]};
      if (cnt < batch) node[cnt++] = {mu[n], h};
    }
    return n;
  }
  // midpoints of the bisection of [lo, hi] whose root is x
  int way(double lo, double hi, double x, double* mu) const {
    int n = 0;
    while (n < batch && (n == 0 || hi - lo > tol)) {
      mu[n] = 0.5 * (lo + hi);
      (mu[n] < x ? lo : hi) = mu[n];
      ++n;
    }
    return n;
  }
};
