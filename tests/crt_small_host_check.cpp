// Host driver for crt_rn where P < 2^96 (at most three 32-bit limbs), as the CRT
// kernel instantiates it there: reads lines "t u_1 ... u_N" and prints, per line,
// whether the path decides the result and its bits.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "oz2_crt_math.h"

namespace {

template <int L>
bool rounded(const oz2::Tables &tab, const int *u, int N, int t, double &r) {
  double acc[L];
  for (int q = 0; q < L; ++q) acc[q] = 0.0;
  for (int l = 0; l < N; ++l)
    for (int q = 0; q < L; ++q) acc[q] = fma(tab.cw[l][q], (double)u[l], acc[q]);
  return oz2::crt_rn<L, true>(acc, tab.cP, tab.inv_P_d, tab.crt_fast, t, r);
}

}  // namespace

int main(int argc, char **argv) {
  if (argc != 3) return 2;
  const int N = atoi(argv[1]), list = atoi(argv[2]);
  static oz2::Tables tab;
  if (!oz2::build_tables(N, list, &tab) || tab.limbs > 3 || tab.wlimbs != tab.limbs) return 3;
  std::vector<int> u(N);
  int t;
  while (scanf("%d", &t) == 1) {
    for (int l = 0; l < N; ++l)
      if (scanf("%d", &u[l]) != 1) return 4;
    double r = 0.0;
    const bool ok = tab.limbs == 1   ? rounded<1>(tab, u.data(), N, t, r)
                    : tab.limbs == 2 ? rounded<2>(tab, u.data(), N, t, r)
                                     : rounded<3>(tab, u.data(), N, t, r);
    uint64_t bits;
    memcpy(&bits, &r, 8);
    printf("%d %016llx\n", ok ? 1 : 0, (unsigned long long)bits);
  }
  return 0;
}
