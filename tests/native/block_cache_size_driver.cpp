// The block cache (block_cache.h) says how large a block is, and what it hands
// out for a size does not depend on what it kept.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "block_cache.h"

static std::map<void *, size_t> size_of;
static size_t budget = ~size_t(0);
static void *take(size_t n) {
  if (n > budget) return nullptr;
  void *p = std::malloc(16);
  size_of[p] = n;
  return p;
}
static void give(void *p) {
  size_of.erase(p);
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
  const size_t limit = size_t(1) << 28;
  sell::BlockCache c(take, give);
  for (size_t n : {size_t(1), size_t(513), size_t(70'000), size_t(1) << 20, (size_t(1) << 20) + 1, limit, limit + 1}) {
    // a kept block of the next two sizes above, which is not for n
    const size_t up = sell::BlockCache::rounded(n) + 1;
    size_t got_cold = 0, got_warm = 0;
    void *a = c.get(0, n, limit, &got_cold);
    CHECK(size_of[a] == got_cold && got_cold >= n && (got_cold - n < 512 || got_cold - n <= n / 16));
    void *larger = up <= limit ? c.get(0, up, limit) : nullptr;
    c.put(0, a, limit, false);
    if (larger) c.put(0, larger, limit);
    void *b = c.get(0, n, limit, &got_warm);
    CHECK(size_of[b] == got_warm && got_warm == got_cold);
    c.put(0, b, limit);
    b = c.get(0, n, limit, &got_warm);
    CHECK(size_of[b] == got_warm && got_warm == got_cold);
    c.put(0, b, limit);
    c.flush();
  }
  budget = 1'000'001;  // only as much as asked for
  size_t got = 0;
  void *p = c.get(0, 1'000'001, limit, &got);
  CHECK(p && got == 1'000'001 && size_of[p] == got);
  c.put(0, p, limit);
  c.flush();
  CHECK(size_of.empty());
  std::puts("ok");
  return 0;
}
