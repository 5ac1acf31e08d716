// Host driver for the CRT kernel's fast path (crt_rn of oz2_crt_math.h) with
// the library's own tables: for N moduli of list `list`, reads lines
// "t u_1 ... u_N" and prints, per line, whether the path decides the result
// and its bits.
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
  return oz2::crt_rn<L>(acc, tab.cP, tab.inv_P_d, tab.crt_fast, t, r);
}

}  // namespace

int main(int argc, char **argv) {
  if (argc != 3) return 2;
  const int N = atoi(argv[1]), list = atoi(argv[2]);
  static oz2::Tables tab;
  if (!oz2::build_tables(N, list, &tab)) return 3;
  std::vector<int> u(N);
  int t;
  while (scanf("%d", &t) == 1) {
    for (int l = 0; l < N; ++l)
      if (scanf("%d", &u[l]) != 1) return 4;
    double r = 0.0;
    bool ok;
    switch (tab.wlimbs) {
      case 1: ok = rounded<1>(tab, u.data(), N, t, r); break;
      case 2: ok = rounded<2>(tab, u.data(), N, t, r); break;
      case 3: ok = rounded<3>(tab, u.data(), N, t, r); break;
      case 4: ok = rounded<4>(tab, u.data(), N, t, r); break;
      case 5: ok = rounded<5>(tab, u.data(), N, t, r); break;
      case 6: ok = rounded<6>(tab, u.data(), N, t, r); break;
      case 7: ok = rounded<7>(tab, u.data(), N, t, r); break;
      case 8: ok = rounded<8>(tab, u.data(), N, t, r); break;
      default: return 5;
    }
    uint64_t bits;
    memcpy(&bits, &r, 8);
    printf("%d %016llx\n", ok ? 1 : 0, (unsigned long long)bits);
  }
  return 0;
}
