// Device memory blocks kept from one matrix for the next. Host code only (no
// HIP), so that it can be checked on its own.
//
// A program that builds a new matrix for every time step frees as many bytes as
// it takes, and freeing a large block is slow: the driver clears it, at about
// 45 GB/s when it has fallen behind (a 27-point stencil of 128^3, 790 MB: up to
// 19 ms of a step that computes for 1). Blocks given back are therefore kept for
// the next construction, within these limits:
//   - at most `limit` bytes and kMaxBlocks blocks altogether (a small block takes a
//     page of device memory whatever its size); the ones kept longest go first,
//     and a block larger than `limit` is freed at once;
//   - a block that kKeep constructions in a row did not use is freed;
//   - when an allocation fails, every kept block of that device is freed and
//     the allocation tried again; flush() frees them all on request.
// Every operation takes the same few steps however many blocks there are: kept
// blocks stand in a list by age and in a stack per size. (One list that was
// searched and shifted: with 15,000 kept blocks a construction spent 0.25 ms here,
// and letting 75,000 go 2.7 s; now 1 us with 4,096, the most there are.) Giving back and
// letting go allocate nothing, so they cannot fail.
// Only a block that is idle is kept, so whoever takes it next may use it on any
// stream: the callers wait for the device first and say whether that succeeded.
// After a wait that was refused (a stream under capture, an earlier error) the
// block is freed, which leaves the waiting to the runtime. A block serves the
// device it was taken on only.
#pragma once

#include <cstddef>
#include <cstdint>
#include <map>
#include <memory>
#include <mutex>
#include <unordered_map>
#include <utility>

namespace sell {

class BlockCache {
 public:
  using Alloc = void *(*)(size_t);  // on the current device; nullptr on failure
  using Free = void (*)(void *);
  BlockCache(Alloc a, Free f) : alloc_(a), free_(f) {}

  static constexpr uint64_t kKeep = 256;  // a batch of matrices may turn over between two uses
  static constexpr size_t kMaxBlocks = 16 * kKeep;  // a construction takes about 15

  // Sizes within a sixteenth of each other share a size, so that matrices of
  // about the same size reuse each other's blocks. A block serves its own size
  // only: what a matrix holds follows from its layout, not from what was kept.
  static size_t rounded(size_t bytes) {
    size_t step = 512;
    while (step * 32 <= bytes) step *= 2;
    return (bytes + step - 1) / step * step;
  }

  // A block of at least `bytes` bytes on `device`, which is the current one; *got
  // (if asked for): its size.
  void *get(int device, size_t bytes, size_t limit, size_t *got = nullptr) {
    const size_t need = bytes <= limit ? rounded(bytes) : bytes;
    if (got) *got = need;
    {
      std::lock_guard<std::mutex> lock(mu_);
      const auto it = sizes_.find({device, need});
      if (it != sizes_.end() && it->second) {
        Block *b = it->second;
        unlink(b);
        return b->p;
      }
    }
    size_t size = need;
    void *p = alloc_(size);
    if (!p) {
      flush(device);
      size = bytes;
      p = alloc_(size);
      if (got) *got = size;
    }
    if (!p) return nullptr;
    try {
      std::unique_ptr<Block> b(new Block{p, size, device});
      std::lock_guard<std::mutex> lock(mu_);
      if (size <= limit && size == rounded(size)) b->stack = &sizes_[{device, size}];
      blocks_[p] = b.get();
      (void)b.release();
    } catch (...) {  // no host memory for the entry
      free_(p);
      p = nullptr;
    }
    return p;
  }

  // Gives p (from get) back. device: the current one; idle: nothing uses p any more.
  void put(int device, void *p, size_t limit, bool idle = true) {
    if (!p) return;
    Block *gone = nullptr;
    {
      std::lock_guard<std::mutex> lock(mu_);
      const auto it = blocks_.find(p);
      if (it == blocks_.end()) return;
      Block *b = it->second;
      if (!idle || b->device != device || b->bytes > limit || !b->stack) {
        let_go(b, &gone);
      } else {
        link(b);
        while (total_ > limit || count_ > kMaxBlocks) {
          Block *o = oldest_;
          unlink(o);
          let_go(o, &gone);
        }
      }
    }
    free_all(gone);
  }

  // A construction ended: frees what kKeep of them have not used.
  void tick() {
    Block *gone = nullptr;
    {
      std::lock_guard<std::mutex> lock(mu_);
      ++epoch_;
      while (oldest_ && oldest_->since + kKeep < epoch_) {
        Block *o = oldest_;
        unlink(o);
        let_go(o, &gone);
      }
    }
    free_all(gone);
  }

  // Frees the kept blocks of a device, or of all (-1); false: there were none.
  bool flush(int device = -1) {
    Block *gone = nullptr;
    {
      std::lock_guard<std::mutex> lock(mu_);
      for (Block *b = oldest_; b;) {
        Block *o = b;
        b = b->younger;
        if (device >= 0 && o->device != device) continue;
        unlink(o);
        let_go(o, &gone);
      }
    }
    const bool any = gone != nullptr;
    free_all(gone);
    return any;
  }

 private:
  struct Block {
    void *p = nullptr;
    size_t bytes = 0;
    int device = 0;
    Block **stack = nullptr;  // top of its size's stack; nullptr: never kept
    uint64_t since = 0;       // the construction count when it was given back
    Block *older = nullptr, *younger = nullptr;  // by age, while kept
    Block *below = nullptr, *above = nullptr;    // in the stack, while kept
  };

  // Into and out of the list and the stack of kept blocks.
  void link(Block *b) {
    b->since = epoch_;
    b->older = youngest_;
    b->younger = nullptr;
    (youngest_ ? youngest_->younger : oldest_) = b;
    youngest_ = b;
    b->below = *b->stack;
    b->above = nullptr;
    if (b->below) b->below->above = b;
    *b->stack = b;
    total_ += b->bytes;
    ++count_;
  }
  void unlink(Block *b) {
    (b->older ? b->older->younger : oldest_) = b->younger;
    (b->younger ? b->younger->older : youngest_) = b->older;
    (b->above ? b->above->below : *b->stack) = b->below;
    if (b->below) b->below->above = b->above;
    total_ -= b->bytes;
    --count_;
  }
  // Takes an unlinked block out of the books and onto the list `gone`: out first,
  // since the driver may hand its address out again as soon as it is freed.
  void let_go(Block *b, Block **gone) {
    blocks_.erase(b->p);
    b->younger = *gone;
    *gone = b;
  }
  void free_all(Block *gone) {
    while (gone) {
      Block *b = gone;
      gone = b->younger;
      free_(b->p);
      delete b;
    }
  }

  Alloc alloc_;
  Free free_;
  std::mutex mu_;
  std::map<std::pair<int, size_t>, Block *> sizes_;  // kept blocks of a device and size, the latest on top
  std::unordered_map<void *, Block *> blocks_;       // all blocks, by address
  Block *oldest_ = nullptr, *youngest_ = nullptr;
  size_t total_ = 0, count_ = 0;
  uint64_t epoch_ = 0;
};

}  // namespace sell
