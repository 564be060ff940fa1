// Host check of the chemical-potential search of the library.
#include "gw_mu.h"
#include <cstdio>

static int bad = 0;
#define CHECK(c)                                            \
  do {                                                      \
    if (!(c)) { ++bad; printf("line %d: %s\n", __LINE__, #c); } \
  } while (0)

// matrices of more than 32 orbitals are inverted one mu after another
static void batch_rule() {
  for (long long m : {2LL, 24LL, 273LL, 274LL, 1000LL, 4096LL, 4097LL, 6400LL, 2048LL * 262144LL})
    for (int nao = 1; nao <= 60; ++nao) {
      const int b = mu_batch(nao, m);
      CHECK(b >= 1 && b <= kMuBatch);
      CHECK(nao <= 32 ? b == 1 || b * m <= 4096 : b == 1);
    }
  CHECK(mu_batch(32, 273) == 15 && mu_batch(32, 1000) == 4 && mu_batch(32, 6400) == 1);
}

int main() {
  batch_rule();
  printf("bad %d\n", bad);
  return bad != 0;
}
