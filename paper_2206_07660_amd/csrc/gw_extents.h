// Host-side proof that the launches of the triple products and of the
// polarization contraction stay inside their operands (GW_DEBUG_BOUNDS).
#pragma once
#include <algorithm>

#include "gw_kernels.h"

// An array: its first element and their number.
struct Arr {
  const void* p;
  long long n;
};

// Offsets, in elements, that a launch touches from an operand's pointer.
struct Reach {
  long long lo = 0, hi = 0;
  Reach& by(long long count, long long stride) {   // + i stride, 0 <= i < count
    lo += std::min(0LL, (count - 1) * stride);
    hi += std::max(0LL, (count - 1) * stride);
    return *this;
  }
  Reach& at(long long least, long long most) {
    lo += least;
    hi += most;
    return *this;
  }
  bool inside(const void* p, long long bytes, Arr a) const {
    const char *q = (const char*)p, *b = (const char*)a.p;
    return q + lo * bytes >= b && q + (hi + 1) * bytes <= b + a.n * bytes;
  }
};

// tab: the host copy of d.tab, whose entries from d.tab on are `entries`.
// Returns the operand that is left, or NULL.
inline const char* sand_prod_leaves(const SandProd& d, const int* tab, long long entries, Arr V, Arr L, Arr R, Arr Y) {
  if (d.nt <= 0 || d.nk <= 0 || d.naux <= 0) return nullptr;
  if (d.nk > entries) return "table";
  const long long n2 = (long long)d.nao * d.nao;
  const long long tl = *std::min_element(tab, tab + d.nk), th = *std::max_element(tab, tab + d.nk);
  const Reach v = Reach().by(d.nk, d.svk).by(d.naux, n2).by(n2, 1);
  auto small = [&](long long ts, int by_tab) {
    Reach r = Reach().by(d.nt, ts).by(n2, 1);
    return by_tab ? r.at(tl * n2, th * n2) : r.by(d.nk, n2);
  };
  if (!v.inside(d.V, 16, V)) return "V";
  if (!small(d.tsL, 0).inside(d.L, 16, L)) return "L";
  if (!small(d.tsR, d.tabR).inside(d.R, 16, R)) return "R";
  if (!Reach(v).by(d.nt, d.tsY).inside(d.Y, 16, Y)) return "Y";
  return nullptr;
}

inline const char* sand_sum_leaves(const SandSum& d, const int* tab, long long entries, Arr A, Arr B, Arr G, Arr O,
                                   Arr part) {
  if (d.nt <= 0 || d.nk <= 0 || d.naux <= 0) return nullptr;
  const long long n2 = (long long)d.nao * d.nao, es = d.tv ? 8 : 16;
  if (d.tstab < 0 || (d.nt - 1) * d.tstab + d.nk > entries) return "table";
  long long tl = tab[0], th = tab[0];
  for (int t = 0; t < d.nt; ++t)
    for (int k = 0; k < d.nk; ++k) {
      tl = std::min(tl, (long long)tab[t * d.tstab + k]);
      th = std::max(th, (long long)tab[t * d.tstab + k]);
    }
  auto small = [&](long long ts, int by_tab) {
    Reach r = Reach().by(d.nt, ts).by(n2, 1);
    return by_tab ? r.at(tl * n2, th * n2) : r.by(d.nk, n2);
  };
  if (!Reach().by(d.nt, d.tsA).by(d.nk, d.skA).by(d.naux, d.sqA).by(n2, 1).inside(d.A, es, A)) return "A";
  if (!Reach().by(d.nt, d.tsB).by(d.nk, d.skB).by(d.naux, d.sqB).by(n2, 1).inside(d.B, es, B)) return "B";
  if (!small(d.tsG, d.tabG).inside(d.G, 16, G)) return "G";
  if (!small(d.fold_t ? 0 : d.tsO, d.tabO).inside(d.O, 16, O)) return "O";
  if (d.part && d.part_elems > 0 && !Reach().by(d.part_elems, 1).inside(d.part, 16, part)) return "part";
  return nullptr;
}

inline const char* pol_acc_leaves(const PolAcc& d, long long part_elems, Arr Y, Arr V, Arr P, Arr M, Arr part) {
  if (d.nt <= 0 || d.naux <= 0 || d.K <= 0) return nullptr;
  const long long n2 = d.n2, nn = (long long)d.naux * d.naux;
  const Reach v = Reach().by(d.K / n2, d.sv).by(d.naux, n2).by(n2, 1);
  if (!Reach(v).by(d.nt, d.tsY).inside(d.Y, 16, Y)) return "Y";
  if (!v.inside(d.V, 16, V)) return "V";
  if (!Reach().by(d.nt, nn).by(nn, 1).inside(d.P, 16, P)) return "P";
  if (d.M && !Reach().by(d.nt, -nn).by(nn, 1).inside(d.M, 16, M)) return "M";
  if (!Reach().by(part_elems, 1).inside(d.part, 16, part)) return "part";
  return nullptr;
}
