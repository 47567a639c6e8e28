// Checks of the block cache (block_cache.h) on the host, memory stood in for
// by malloc with a budget. Prints "ok", or what failed, and exits accordingly.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <thread>
#include <vector>

#include "block_cache.h"

static std::mutex mu;
static std::map<void *, size_t> held;
static size_t in_use = 0, budget = ~size_t(0);
static long allocs = 0, frees = 0;

static void *take(size_t n) {
  std::lock_guard<std::mutex> l(mu);
  if (in_use + n > budget) return nullptr;
  void *p = std::malloc(16);
  held[p] = n;
  in_use += n;
  ++allocs;
  return p;
}

static void give(void *p) {
  std::lock_guard<std::mutex> l(mu);
  const auto it = held.find(p);
  if (it == held.end()) {
    std::puts("freed twice");
    std::exit(1);
  }
  in_use -= it->second;
  held.erase(it);
  std::free(p);
  ++frees;
}

#define CHECK(c)                                    \
  do {                                              \
    if (!(c)) {                                     \
      std::printf("line %d: %s\n", __LINE__, #c);   \
      return 1;                                     \
    }                                               \
  } while (0)

int main() {
  const size_t MB = 1 << 20, limit = 100 * MB;
  sell::BlockCache c(take, give);
  // sizes: never smaller than asked, at most a sixteenth more
  for (size_t n : {size_t(1), size_t(511), size_t(512), size_t(100'000), 3 * MB + 1, 450 * MB + 7}) {
    const size_t r = sell::BlockCache::rounded(n);
    CHECK(r >= n && (r - n < 512 || r - n <= n / 16));
  }
  // a block of the same size class comes back, one of another size does not
  void *a = c.get(0, 10 * MB, limit);
  c.put(0, a, limit);
  CHECK(c.get(0, 10 * MB - 5, limit) == a && allocs == 1);
  c.put(0, a, limit);
  void *b = c.get(0, 30 * MB, limit);
  CHECK(b != a && allocs == 2);
  // not on another device; put back under another device: freed
  void *d = c.get(1, 10 * MB, limit);
  CHECK(d != a && allocs == 3);
  c.put(0, d, limit);
  CHECK(frees == 1);
  // the limit: the oldest goes; larger than the limit: freed at once
  c.put(0, b, limit);
  void *e = c.get(0, 80 * MB, limit);
  c.put(0, e, limit);
  CHECK(in_use <= limit && frees == 3);  // a, b
  void *f = c.get(0, 200 * MB, limit);
  c.put(0, f, limit);
  CHECK(frees == 4 && in_use <= limit);
  // unused for kKeep constructions
  for (uint64_t i = 0; i <= sell::BlockCache::kKeep; ++i) {
    CHECK(in_use > 0);
    c.tick();
  }
  CHECK(in_use == 0);
  // a failing allocation takes the kept blocks first
  budget = 100 * MB;
  void *g = c.get(0, 60 * MB, limit);
  c.put(0, g, limit);
  void *h = c.get(0, 90 * MB, limit);
  CHECK(h && in_use <= budget && !c.get(0, 60 * MB, limit));
  c.put(0, h, limit);
  c.flush();
  CHECK(in_use == 0);
  // threads: no block is handed out twice
  budget = ~size_t(0);
  std::mutex own_mu;
  std::map<void *, int> own;
  std::atomic<int> bad{0};
  std::vector<std::thread> ts;
  for (int t = 0; t < 8; ++t)
    ts.emplace_back([&, t] {
      unsigned s = (unsigned)t + 1;
      for (int i = 0; i < 3000; ++i) {
        s = s * 1664525u + 1013904223u;
        void *p = c.get(t & 1, (1 + s % 40) * MB / 4, limit);
        {
          std::lock_guard<std::mutex> l(own_mu);
          if (!own.emplace(p, t).second) ++bad;
        }
        {
          std::lock_guard<std::mutex> l(own_mu);
          own.erase(p);
        }
        c.put(t & 1, p, limit);
        if (i % 7 == 0) c.tick();
      }
    });
  for (auto &t : ts) t.join();
  CHECK(bad == 0 && in_use <= limit);
  c.flush();
  CHECK(in_use == 0 && allocs == frees);
  std::puts("ok");
  return 0;
}
