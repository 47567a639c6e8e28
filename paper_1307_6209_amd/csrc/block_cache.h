// Device memory blocks kept from one matrix for the next. Host code only (no
// HIP), so that it can be checked on its own.
//
// A program that builds a new matrix for every time step frees as many bytes as
// it takes, and freeing a large block is slow: the driver clears it, at about
// 45 GB/s when it has fallen behind (a 27-point stencil of 128^3, 790 MB: up to
// 19 ms of a step that computes for 1). Blocks given back are therefore kept for
// the next construction, within these limits:
//   - at most `limit` bytes altogether; the ones kept longest go first, and
//     a block larger than that is freed at once;
//   - a block that kKeep constructions in a row did not use is freed;
//   - when an allocation fails, every kept block of that device is freed and
//     the allocation tried again; flush() frees them all on request.
// Only a block that is idle is kept, so whoever takes it next may use it on any
// stream: the callers wait for the device first and say whether that succeeded.
// After a wait that was refused (a stream under capture, an earlier error) the
// block is freed, which leaves the waiting to the runtime. A block serves the
// device it was taken on only.
#pragma once

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace sell {

class BlockCache {
 public:
  using Alloc = void *(*)(size_t);  // on the current device; nullptr on failure
  using Free = void (*)(void *);
  BlockCache(Alloc a, Free f) : alloc_(a), free_(f) {}

  static constexpr uint64_t kKeep = 256;  // a batch of matrices may turn over between two uses

  // Sizes within a sixteenth of each other share a size, so that matrices of
  // about the same size reuse each other's blocks.
  static size_t rounded(size_t bytes) {
    size_t step = 512;
    while (step * 32 <= bytes) step *= 2;
    return (bytes + step - 1) / step * step;
  }

  // A block of at least `bytes` bytes on `device`, which is the current one.
  void *get(int device, size_t bytes, size_t limit) {
    const size_t need = bytes <= limit ? rounded(bytes) : bytes;
    {
      std::lock_guard<std::mutex> lock(mu_);
      size_t best = kept_.size();
      for (size_t i = 0; i < kept_.size(); ++i)
        if (kept_[i].device == device && kept_[i].bytes >= need && kept_[i].bytes <= need + need / 8 &&
            (best == kept_.size() || kept_[i].bytes < kept_[best].bytes))
          best = i;
      if (best < kept_.size()) {
        Block b = kept_[best];
        kept_.erase(kept_.begin() + (ptrdiff_t)best);
        total_ -= b.bytes;
        used_[b.p] = b;
        return b.p;
      }
    }
    size_t size = need;
    void *p = alloc_(size);
    if (!p) {
      flush(device);
      size = bytes;
      p = alloc_(size);
    }
    if (!p) return nullptr;
    try {
      std::lock_guard<std::mutex> lock(mu_);
      used_[p] = Block{p, size, device, 0};
    } catch (...) {  // no host memory for the entry
      free_(p);
      p = nullptr;
    }
    return p;
  }

  // Gives p (from get) back. device: the current one; idle: nothing uses p any more.
  void put(int device, void *p, size_t limit, bool idle = true) {
    if (!p) return;
    std::vector<void *> gone;
    {
      std::lock_guard<std::mutex> lock(mu_);
      const auto it = used_.find(p);
      if (it == used_.end()) return;
      Block b = it->second;
      used_.erase(it);
      if (!idle || b.device != device || b.bytes > limit) {
        gone.push_back(p);
      } else {
        b.since = epoch_;
        kept_.push_back(b);
        total_ += b.bytes;
        while (total_ > limit) take_out(0, gone);  // the front was given back first
      }
    }
    for (void *q : gone) free_(q);
  }

  // A construction ended: frees what kKeep of them have not used.
  void tick() {
    std::vector<void *> gone;
    {
      std::lock_guard<std::mutex> lock(mu_);
      ++epoch_;
      for (size_t i = 0; i < kept_.size();) {
        if (kept_[i].since + kKeep < epoch_) take_out(i, gone);
        else ++i;
      }
    }
    for (void *q : gone) free_(q);
  }

  // Frees the kept blocks of a device, or of all (-1); false: there were none.
  bool flush(int device = -1) {
    std::vector<void *> gone;
    {
      std::lock_guard<std::mutex> lock(mu_);
      for (size_t i = 0; i < kept_.size();) {
        if (device < 0 || kept_[i].device == device) take_out(i, gone);
        else ++i;
      }
    }
    for (void *q : gone) free_(q);
    return !gone.empty();
  }

 private:
  struct Block {
    void *p;
    size_t bytes;
    int device;
    uint64_t since;  // the construction count when it was given back
  };
  void take_out(size_t i, std::vector<void *> &gone) {
    gone.push_back(kept_[i].p);
    total_ -= kept_[i].bytes;
    kept_.erase(kept_.begin() + (ptrdiff_t)i);
  }

  Alloc alloc_;
  Free free_;
  std::mutex mu_;
  std::vector<Block> kept_;  // in the order they were given back
  std::unordered_map<void *, Block> used_;
  size_t total_ = 0;
  uint64_t epoch_ = 0;
};

}  // namespace sell
