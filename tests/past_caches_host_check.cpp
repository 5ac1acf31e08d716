// Prints, for lines "megabytes whole_lines batch", whether a C of that size is stored
// past the caches.
#include <stdio.h>

#include "oz2_internal.h"

int main() {
  long long mb;
  int whole, batch;
  while (scanf("%lld %d %d", &mb, &whole, &batch) == 3)
    printf("%d\n", oz2::past_caches(mb << 20, whole != 0, batch != 0) ? 1 : 0);
  return 0;
}
