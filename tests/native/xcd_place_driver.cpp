// Host driver of xcd_place (xcd_place.h): reads n, workgroup size and number of
// XCDs, prints the place of each unit.
#include <cstdio>

#include "xcd_place.h"

int main() {
  long long n, W, X;
  if (std::scanf("%lld %lld %lld", &n, &W, &X) != 3) return 2;
  for (long long k = 0; k < n; ++k) std::printf("%lld ", (long long)sell::xcd_place(k, n, (int)W, (int)X));
  return 0;
}
