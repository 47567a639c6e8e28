// Host driver of the block form's choice between one pass of any width and the pass
// kernel (block_rule.h): lines of C k local padded longest, answered by
// "kv passes lanes pairs wins".
#include <cstdio>

#include "block_rule.h"

int main() {
  long long C, k, local, padded, longest;
  while (std::scanf("%lld %lld %lld %lld %lld", &C, &k, &local, &padded, &longest) == 5) {
    const int rpw = C < 64 ? (int)C : 64, kv = sell::pass_width(rpw, (int)k, 0);
    const int width = 64 / rpw * kv, passes = ((int)k + width - 1) / width;
    const int lanes = sell::spmmv_any_lanes((int)C, (int)k, local != 0);
    const int pairs = ((int)k + 2 * lanes - 1) / (2 * lanes);
    const bool wins = passes > 1 && sell::one_pass_wins(padded, longest, rpw, lanes, pairs, kv, passes);
    std::printf("%d %d %d %d %d\n", kv, passes, lanes, pairs, wins ? 1 : 0);
  }
  return 0;
}
