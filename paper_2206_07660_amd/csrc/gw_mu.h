// Host side of the chemical-potential search (internal).
#pragma once
#include <algorithm>
#include <cmath>

#include "../../include/gw.h"

constexpr int kMuBatch = 15;   // most values of mu in one launch

// Counts that a launch of the search takes: all of the next levels, or one way
// ahead.
struct MuCounts {
  int batch, ahead;
};

// For `matrices` = nw_f nk Dyson matrices of order nao.  A launch costs about
// 17 us beside its counts; a count costs about 22.5 ps nao^2 per matrix (6400 of
// them: 13 us at nao 8, 31 at 16, 103 at 26, 148 at 32, 5 of these the launch's),
// so that the levels of a tree of b counts, log2(b + 1), are worth b of them up
// to 1 / 2.5 / 8 us per count for b = 15 / 7 / 3.  Counts ahead are wasted only
// where the way is left, about every third one in a gap, which launches outweigh
// up to 16 us.  Matrices of more than 32 orbitals are inverted one value of mu
// after another, so a second value costs as much as the first.
inline MuCounts mu_counts(int nao, long long matrices) {
  if (nao > 32) return {1, 1};
  const double us = 22.5e-6 * nao * nao * (double)matrices;
  const int room = (int)std::max(1LL, 262144LL / matrices);   // partial sums: 2 MB
  const int batch = std::min(room, us <= 1.0 ? kMuBatch : us <= 2.5 ? 7 : us <= 8.0 ? 3 : 1);
  return {batch, us <= 16.0 ? std::min(room, kMuBatch) : batch};
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
// order of the midpoints picks one.  A launch takes all midpoints of the next
// levels (batch counts) or, where the secant's root of the bracket agrees with
// that of the bracket before, the first midpoints on the way to it (up to ahead
// counts; where the secants converge each such launch doubles the known digits).
// Counts that the plain bisection would not have asked for decide nothing.
// One search to 1e-13 is 47 counts; in launches of
//   15 / 15 counts  58 .. 110 of them in 6 .. 10 launches (metal), 140 .. 180 in 11 .. 14 (gap)
//    3 / 15         48 .. 63 in 5 .. 11, 67 .. 85 in 14 .. 26
//    1 / 15         47 .. 60 in 6 .. 16, 55 .. 73 in 16 .. 41
// (metal / gap).  Times: 2x2x2, nao 6, 24 frequencies 0.20 / 0.24 ms, 3x3x3, nao
// 16, 60 0.62 / 1.16, 4x4x4, nao 26, 100 5.4 / 5.4; 1.9, 3.8 and 16.9 ms with
// one workgroup-wide inversion and one copied count at a time.  Taking
// counts to rise with mu, and skipping the midpoints that this settles, gives
// 0.20 / 0.34, 0.43 / 1.5 and 1.9 / 5.9 ms, but has moved mu by 0.2 Ha in a gap
// (beta 1000, 24 nodes).
//
// at(mu, n, ne) forms the counts ne[i] at mu[i], i < n <= max(batch, ahead).
template <class Count>
struct MuRoot {
  Count at;
  int batch, ahead;
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
    double before = lo;                       // the secant's root in the bracket before
    int cap = ahead;
    for (int it = 0; hi - lo > tol && it < 400;) {
      // the secant's root, and the levels down to which it agrees with the one
      // before: the bisection goes its way at least that far as a rule, and
      // about twice as far where the secants converge
      const double x = lo + (hi - lo) * ((target - nlo) / (nhi - nlo));
      const double ratio = (hi - lo) / std::fabs(x - before);
      const int levels = ratio >= 2.0 ? std::ilogb(std::min(ratio, 1e9)) : 0;
      before = x;
      double mu[kMuBatch], ne[kMuBatch];
      const bool follow = (1 << std::min(levels, cap)) > batch;
      const int n = follow ? way(lo, hi, x, std::min(2 * levels, cap), mu) : tree(lo, hi, mu), it0 = it;
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
      // rounding makes secants agree as well: a way that was left is not
      // followed as far again at once
      if (x < lo || x > hi) cap = follow ? std::max(1, (it - it0) / 2) : cap;
      else cap = std::min(ahead, 2 * cap);
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
  // the first midpoints of the bisection of [lo, hi] whose root is x
  int way(double lo, double hi, double x, int most, double* mu) const {
    int n = 0;
    while (n < most && (n == 0 || hi - lo > tol)) {
      mu[n] = 0.5 * (lo + hi);
      (mu[n] < x ? lo : hi) = mu[n];
      ++n;
    }
    return n;
  }
};
