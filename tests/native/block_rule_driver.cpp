// Host driver of the block form's rule (block_rule.h): lines of
// C group nchunks padded maxwin maxseg runs lds cus k, answered by
// "kb turns" (0 0: the other kernels).
#include <cstdio>

#include "block_rule.h"

int main() {
  long long C, group, nchunks, padded, maxwin, maxseg, runs, lds, cus, k;
  while (std::scanf("%lld %lld %lld %lld %lld %lld %lld %lld %lld %lld", &C, &group, &nchunks, &padded, &maxwin,
                    &maxseg, &runs, &lds, &cus, &k) == 10) {
    const sell::BlockTurns t = sell::block_turns(
        sell::block_windows((int)C, (int)group, nchunks, padded, (int)maxwin, (int)maxseg, runs, (size_t)lds, (int)cus),
        (int)k);
    std::printf("%d %d\n", t.kb, t.turns);
  }
  return 0;
}
