// Host check of the extents that GW_DEBUG_BOUNDS proves for the launches of the
// triple products and the polarization contraction: every offset of the formulas
// in gw_kernels.h, walked one by one, against the arrays found to be enough.
#include "gw_extents.h"
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

static int bad = 0;
#define CHECK(c)                                                \
  do {                                                          \
    if (!(c)) { ++bad; printf("line %d: %s\n", __LINE__, #c); } \
  } while (0)

static uint64_t seed = 88172645463325252ull;
static int rnd(int a, int b) {   // a..b
  seed ^= seed << 13; seed ^= seed >> 7; seed ^= seed << 17;
  return a + (int)(seed % (uint64_t)(b - a + 1));
}

// first and last offset of a walk
struct Walk {
  bool any = false;
  long long lo = 0, hi = 0;
  void at(long long o) {
    lo = any ? std::min(lo, o) : o;
    hi = any ? std::max(hi, o) : o;
    any = true;
  }
};

// p: base of one big allocation; operand o starts at p + at[o], its array spans the walk exactly
struct Op {
  const char* p;
  Walk w;
  long long es;
  Arr fit(int cut_lo, int cut_hi) const { return Arr{p + (w.lo + cut_lo) * es, w.hi - w.lo + 1 - cut_lo - cut_hi}; }
};

static char room[1];

// check(arrays) must accept the exact arrays and name the operand whose array is one element short
template <class F> static void tight(std::vector<Op>& ops, const std::vector<const char*>& names, F check) {
  auto arrs = [&](int which, int lo, int hi) {
    std::vector<Arr> a;
    for (int i = 0; i < (int)ops.size(); ++i) a.push_back(ops[i].fit(i == which ? lo : 0, i == which ? hi : 0));
    return a;
  };
  CHECK(check(arrs(-1, 0, 0)) == nullptr);
  for (int i = 0; i < (int)ops.size(); ++i)
    for (int side = 0; side < 2; ++side) {
      const char* r = check(arrs(i, side, 1 - side));
      CHECK(r && !std::strcmp(r, names[i]));
    }
}

int main() {
  for (int it = 0; it < 400; ++it) {
    const int nt = rnd(1, 4), nk = rnd(1, 5), naux = rnd(1, 4), nao = rnd(1, 3), n2 = nao * nao, q = rnd(0, nk - 1);
    const long long sv = (long long)naux * n2 + (it % 3 == 0 ? 5 : 0), gs = (long long)nk * n2, S = nk * sv;
    std::vector<int> plus((size_t)nk * nk);
    for (auto& x : plus) x = rnd(0, nk - 1);
    const int* tab = plus.data() + (size_t)q * nk;
    const long long left = (long long)plus.size() - (long long)q * nk;
    auto sign = [&]() { return rnd(0, 1) ? 1 : -1; };
    // operands far apart: only their own offsets count
    const char* base = room;
    auto op = [&](int i, int es) { return Op{base + i * 100000000LL, Walk{}, es}; };
    {
      SandProd d{};
      std::vector<Op> o{op(1, 16), op(2, 16), op(3, 16), op(4, 16)};
      d.V = (const double2*)o[0].p; d.L = (const double2*)o[1].p; d.R = (const double2*)o[2].p; d.Y = (double2*)o[3].p;
      d.nt = nt; d.nk = nk; d.naux = naux; d.nao = nao; d.svk = sv;
      d.tsL = sign() * gs; d.tsR = sign() * gs; d.tsY = S; d.tabR = rnd(0, 1);
      for (int t = 0; t < nt; ++t)
        for (int k = 0; k < nk; ++k)
          for (int e = 0; e < n2; ++e) {
            o[1].w.at(t * d.tsL + (long long)k * n2 + e);
            o[2].w.at(t * d.tsR + (long long)(d.tabR ? tab[k] : k) * n2 + e);
            for (int Q = 0; Q < naux; ++Q) {
              o[0].w.at(k * sv + (long long)Q * n2 + e);
              o[3].w.at(t * d.tsY + k * sv + (long long)Q * n2 + e);
            }
          }
      tight(o, {"V", "L", "R", "Y"}, [&](const std::vector<Arr>& a) {
        return sand_prod_leaves(d, tab, left, a[0], a[1], a[2], a[3]);
      });
      CHECK(!std::strcmp(sand_prod_leaves(d, tab, nk - 1, o[0].fit(0, 0), o[1].fit(0, 0), o[2].fit(0, 0), o[3].fit(0, 0)), "table"));
      d.nt = 0;
      CHECK(!sand_prod_leaves(d, tab, left, Arr{}, Arr{}, Arr{}, Arr{}));
    }
    {
      SandSum d{};
      d.tv = rnd(0, 1);
      const int es = d.tv ? 8 : 16;
      std::vector<Op> o{op(1, es), op(2, es), op(3, 16), op(4, 16), op(5, 16)};
      d.A = o[0].p; d.B = o[1].p; d.G = (const double2*)o[2].p; d.O = (double2*)o[3].p; d.part = (double2*)o[4].p;
      d.nt = rnd(0, 1) ? std::min(nt, nk - q) : nt;
      d.tstab = d.nt <= nk - q && rnd(0, 1) ? nk : 0;
      d.nk = nk; d.naux = naux; d.nao = nao;
      d.tsA = rnd(0, 1) * S; d.skA = sv; d.sqA = n2;
      d.tsB = S; d.skB = rnd(0, 1) ? sv : n2; d.sqB = d.skB == sv ? n2 : gs;
      // (a table of its own per t: the small matrices do not move with t, as in the exchange)
      d.tsG = d.tstab ? 0 : sign() * gs; d.tsO = d.tstab ? 0 : sign() * gs; d.tabG = rnd(0, 1); d.tabO = rnd(0, 1);
      d.fold_t = rnd(0, 1); d.part_elems = rnd(1, 50);
      for (int t = 0; t < d.nt; ++t)
        for (int k = 0; k < nk; ++k)
          for (int e = 0; e < n2; ++e) {
            const int kq = tab[t * d.tstab + k];
            o[2].w.at(t * d.tsG + (long long)(d.tabG ? kq : k) * n2 + e);
            o[3].w.at((d.fold_t ? 0 : t * d.tsO) + (long long)(d.tabO ? kq : k) * n2 + e);
            for (int Q = 0; Q < naux; ++Q) {
              o[0].w.at(t * d.tsA + k * d.skA + Q * d.sqA + e);
              o[1].w.at(t * d.tsB + k * d.skB + Q * d.sqB + e);
            }
          }
      for (long long e = 0; e < d.part_elems; ++e) o[4].w.at(e);
      auto call = [&](const std::vector<Arr>& a) { return sand_sum_leaves(d, tab, left, a[0], a[1], a[2], a[3], a[4]); };
      tight(o, {"A", "B", "G", "O", "part"}, call);
      CHECK(!std::strcmp(sand_sum_leaves(d, tab, (d.nt - 1) * d.tstab + nk - 1, Arr{}, Arr{}, Arr{}, Arr{}, Arr{}), "table"));
    }
    {
      PolAcc d{};
      std::vector<Op> o{op(1, 16), op(2, 16), op(3, 16), op(4, 16), op(5, 16)};
      d.Y = (const double2*)o[0].p; d.V = (const double2*)o[1].p; d.P = (double2*)o[2].p; d.M = (double2*)o[3].p;
      d.part = (double2*)o[4].p;
      d.nt = nt; d.naux = naux; d.n2 = n2; d.K = nk * n2; d.tsY = S; d.sv = sv;
      const long long elems = rnd(1, 60), nn = (long long)naux * naux;
      for (int t = 0; t < nt; ++t) {
        for (int k = 0; k < nk; ++k)
          for (int Q = 0; Q < naux; ++Q)
            for (int e = 0; e < n2; ++e) {
              o[0].w.at(t * S + k * sv + (long long)Q * n2 + e);
              o[1].w.at(k * sv + (long long)Q * n2 + e);
            }
        for (long long e = 0; e < nn; ++e) {
          o[2].w.at(t * nn + e);
          o[3].w.at(-t * nn + e);
        }
      }
      for (long long e = 0; e < elems; ++e) o[4].w.at(e);
      tight(o, {"Y", "V", "P", "M", "part"}, [&](const std::vector<Arr>& a) {
        return pol_acc_leaves(d, elems, a[0], a[1], a[2], a[3], a[4]);
      });
      d.M = nullptr;
      CHECK(!pol_acc_leaves(d, elems, o[0].fit(0, 0), o[1].fit(0, 0), o[2].fit(0, 0), Arr{}, o[4].fit(0, 0)));
    }
  }
  printf("bad %d\n", bad);
  return bad != 0;
}
