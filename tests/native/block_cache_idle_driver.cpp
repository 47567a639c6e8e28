// The block cache (block_cache.h) keeps idle blocks only: one given back after a
// wait that failed is freed at once and never handed out again.
#include <cstdio>
#include <cstdlib>

#include "block_cache.h"

static long allocs = 0, frees = 0;
static void *take(size_t) {
  ++allocs;
  return std::malloc(16);
}
static void give(void *p) {
  ++frees;
  std::free(p);
}

#define CHECK(c)                                    \
  do {                                              \
    if (!(c)) {                                     \
      std::printf("line %d: %s\n", __LINE__, #c);   \
      return 1;                                     \
    }                                               \
  } while (0)

int main() {
  const size_t limit = size_t(1) << 30;
  sell::BlockCache c(take, give);
  void *a = c.get(0, 1 << 20, limit);
  c.put(0, a, limit, false);
  CHECK(frees == 1 && !c.flush());  // nothing kept
  void *b = c.get(0, 1 << 20, limit);
  CHECK(allocs == 2);
  c.put(0, b, limit, true);
  CHECK(frees == 1 && c.get(0, 1 << 20, limit) == b && allocs == 2);
  std::puts("ok");
  return 0;
}
