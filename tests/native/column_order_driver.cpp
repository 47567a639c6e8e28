// Host driver of order_by_column (batch_plan.h) for the CPU tests: reads
// nunits waves_per_block xcds  and nunits columns; prints the order.
#include <cstdio>
#include <vector>

#include "batch_plan.h"

int main() {
  long long n, W, X;
  if (std::scanf("%lld %lld %lld", &n, &W, &X) != 3) return 2;
  std::vector<int32_t> rep((size_t)n);
  for (auto &r : rep) {
    long long c;
    if (std::scanf("%lld", &c) != 1) return 2;
    r = (int32_t)c;
  }
  for (int32_t v : sell::order_by_column(rep, (int)W, (int)X)) std::printf("%d ", v);
  return 0;
}
