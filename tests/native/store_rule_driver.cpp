// Host driver of the rule for stores of y (store_rule.h): lines of rows, size of an
// element of y, columns, of x, padded slots, of a value, occupancy; 1: through the L2.
#include <cstdio>

#include "store_rule.h"

int main() {
  long long n, ys, m, xs, padded, vs;
  double beta;
  while (std::scanf("%lld %lld %lld %lld %lld %lld %lf", &n, &ys, &m, &xs, &padded, &vs, &beta) == 7)
    std::printf("%d\n", sell::keeps_y(n, (size_t)ys, m, (size_t)xs, padded, (size_t)vs, beta) ? 1 : 0);
  return 0;
}
