// Host side of the chemical-potential search (internal).
#pragma once
#include <algorithm>

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
