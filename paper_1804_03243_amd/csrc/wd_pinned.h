// Pinned host memory that result downloads land in (one pool per device), apart
// from the calls that allocate it so that its rules can be checked on the host.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <memory>
#include <mutex>

namespace wd {

// A call with results of some size leases a block, the copy engine writes its
// results there, and they are viewed in place: the block goes back when the last
// result of the call is freed.  (Copied into vectors, a batch's 25 MB of results
// cost 6 ms of page faults and copies, a wide lattice's 70 MB 20 ms.)  Small
// results, and those of a program that keeps all blocks, go through one block
// that is never leased and are copied out of it: DMA into pageable memory costs
// more than DMA and a copy.  At most kPinnedBlocks + 1 blocks of at most
// kPinnedMax bytes each; a block is kept for the next call, and given back to
// the system where a larger one takes its place.
constexpr int kPinnedBlocks = 3;
constexpr uint64_t kPinnedMax = 512ull << 20;
constexpr uint64_t kPinnedMin = 1ull << 20;
// Results up to this size are copied out at once, so that a program that keeps
// them does not keep a block (64 KB: below malloc's own mappings, some 10 µs).
constexpr uint64_t kPinnedSmall = 64ull << 10;

// Host: static char* alloc(uint64_t bytes) (null when there is none) and
// static void release(char*).
template <class Host>
class PinnedPool {
  struct Block {
    char* p = nullptr;
    uint64_t cap = 0;
    bool leased = false;
  };

 public:
  // A leased block; gives it back when the last holder is gone.
  class Lease {
   public:
    Lease(PinnedPool* pool, Block* block) : pool_(pool), block_(block) {}
    Lease(const Lease&) = delete;
    Lease& operator=(const Lease&) = delete;
    ~Lease() { pool_->give_back(block_); }
    char* data() const { return block_->p; }

   private:
    PinnedPool* pool_;
    Block* block_;
  };

  // A block of at least `bytes`, or null when none is free, the size is beyond
  // the pool's, or no memory can be pinned.
  std::shared_ptr<Lease> lease(uint64_t bytes) {
    if (bytes > kPinnedMax) return nullptr;
    Block* best = nullptr;  // a free block: the smallest that holds the bytes, else the largest
    {
      std::lock_guard<std::mutex> lk(mu_);
      for (Block& b : block_) {
        if (b.leased) continue;
        if (!best || (b.cap >= bytes ? best->cap < bytes || b.cap < best->cap : best->cap < bytes && b.cap > best->cap))
          best = &b;
      }
      if (!best) return nullptr;
      best->leased = true;
    }
    // (allocated outside the lock: it takes milliseconds)
    if (!fit(*best, bytes)) {
      give_back(best);
      return nullptr;
    }
    return std::make_shared<Lease>(this, best);
  }

  // The block that is never leased, for whoever holds stage_lock; null when it
  // cannot hold `bytes`.
  std::mutex& stage_lock() { return stage_mu_; }
  char* stage(uint64_t bytes) { return bytes <= kPinnedMax && fit(stage_, bytes) ? stage_.p : nullptr; }

 private:
  static bool fit(Block& b, uint64_t bytes) {
    if (b.cap >= bytes) return true;
    if (b.p) Host::release(b.p);
    b.p = nullptr;
    b.cap = 0;
    const uint64_t want = std::min(std::max(bytes + bytes / 4, kPinnedMin), kPinnedMax);
    b.p = Host::alloc(want);
    if (b.p) b.cap = want;
    return b.p != nullptr;
  }
  void give_back(Block* b) {
    std::lock_guard<std::mutex> lk(mu_);
    b->leased = false;
  }

  std::mutex mu_, stage_mu_;
  Block block_[kPinnedBlocks], stage_;
};

}  // namespace wd
