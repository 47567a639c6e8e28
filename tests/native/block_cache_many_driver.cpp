// The block cache (block_cache.h) with many small blocks: their number is
// bounded, no operation's cost grows with it, and giving back needs no host
// memory.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <unordered_set>
#include <vector>

#include "block_cache.h"

static bool no_memory = false;
void *operator new(size_t n) {
  void *p = no_memory ? nullptr : std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

static long live = 0;
static void *take(size_t) {
  ++live;
  return std::malloc(16);
}
static void give(void *p) {
  --live;
  std::free(p);
}

#define CHECK(c)                                    \
  do {                                              \
    if (!(c)) {                                     \
      std::printf("line %d: %s\n", __LINE__, #c);   \
      return 1;                                     \
    }                                               \
  } while (0)

static double now() {
  return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

int main() {
  const size_t limit = size_t(4) << 30;
  const long most = (long)sell::BlockCache::kMaxBlocks;
  sell::BlockCache c(take, give);
  // 75,000 blocks of 5,000 small matrices given back: a bounded number is kept
  std::vector<void *> held;
  for (int i = 0; i < 75000; ++i) held.push_back(c.get(0, 300 + (size_t)(i % 997) * 512, limit));
  for (void *p : held) c.put(0, p, limit);
  CHECK(live > 0 && live <= most);
  // the youngest stay
  CHECK(c.get(0, 300 + (size_t)(74999 % 997) * 512, limit) == held.back());
  c.put(0, held.back(), limit);
  // each of them handed out once, by size
  std::unordered_set<void *> seen;
  std::vector<void *> again;
  const long before = live;
  for (int i = 74999; i > 74999 - before; --i) {
    void *p = c.get(0, 300 + (size_t)(i % 997) * 512, limit);
    CHECK(seen.insert(p).second);
    again.push_back(p);
  }
  CHECK(live == before);
  // without host memory: blocks still go back, age out and are freed; a new one is refused, not lost
  no_memory = true;
  for (void *p : again) c.put(0, p, limit);
  CHECK(c.get(0, 900 * 512, limit) != nullptr);
  void *none = c.get(0, size_t(1) << 30, limit);
  no_memory = false;
  CHECK(!none && live == before);
  const double t0 = now();
  for (uint64_t i = 0; i <= sell::BlockCache::kKeep; ++i) c.tick();
  CHECK(live == 1);  // the one handed out last
  // a construction's 15 blocks among as many kept ones as there may be
  held.clear();
  for (long i = 0; i < most; ++i) held.push_back(c.get(0, (size_t)(1 + i) * 4096, limit));
  for (void *p : held) c.put(0, p, limit);
  for (int i = 0; i < 20000; ++i) {
    void *p[15];
    for (int q = 0; q < 15; ++q) p[q] = c.get(0, (size_t)(1 + (i * 15 + q) % 40) * 4096, limit);
    for (int q = 0; q < 15; ++q) c.put(0, p[q], limit);
  }
  const double us = (now() - t0) / 20000 * 1e6;
  std::fprintf(stderr, "%.2f us a construction\n", us);
  std::printf("%s\n", us < 100 ? "ok" : "slow");
  return us < 100 ? 0 : 1;
}
