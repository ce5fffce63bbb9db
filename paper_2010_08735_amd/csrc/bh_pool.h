// Idle device blocks kept for reuse.  Plain C++17, no HIP: the device is a template argument (the
// HIP one in libbh.cpp; a scripted one in the CPU tests) with
//   bool alloc(void** p, size_t bytes), void free(void* p), bool wait()
// where wait() returns true once no work queued so far, on any stream, can use any block.
//
// Fresh device memory is cleared before a process gets it, and a build that allocates and frees a
// 268 MB map waits for that: a new 6 x 2048^2 star map took 4.5 ms of which its kernels are 0.35.
// So idle blocks of at least kKeepLeast are kept, at most kKeepMost in all, and handed out again
// by size.  Past kKeepMost a block makes room when it was not asked for during the last kStale
// calls, so that sizes of the past do not fill the pool for good; builds that need more in all
// than is kept still find what is.  (Room made for every block: the maps of 10^7 stars on 6 x
// 4096^2, 1 GiB each, and their scratch put each other out, 3.19 ms a build for 2.77.)  Sizes are
// rounded up to eight steps an octave so that nearly equal builds share blocks.  Kept blocks are
// freed with the pool's owner, and all pools of a device (Peers) free theirs when an allocation on
// it fails, before it is tried again.
#pragma once

#include <cstddef>
#include <iterator>
#include <list>
#include <mutex>
#include <set>

namespace bh {

constexpr size_t kKeepLeast = (size_t)1 << 20, kKeepMost = (size_t)1 << 30;
constexpr unsigned kStale = 64;

template <class Device>
class BlockPool {
 public:
  // The pools of one device.
  class Peers {
   public:
    void drop() {
      std::lock_guard<std::mutex> g(mu_);
      for (BlockPool* p : pools_) p->drop();
    }

   private:
    friend class BlockPool;
    std::mutex mu_;  // held before a pool's own
    std::set<BlockPool*> pools_;
  };

  BlockPool(Device d, Peers& peers) : dev_(d), peers_(peers) {
    std::lock_guard<std::mutex> g(peers_.mu_);
    peers_.pools_.insert(this);
  }
  ~BlockPool() {
    std::lock_guard<std::mutex> g(peers_.mu_);
    peers_.pools_.erase(this);
  }
  BlockPool(const BlockPool&) = delete;

  // `keeps`: false allocates and frees exactly what is asked for, and keeps nothing (a context
  // whose budget counts what is allocated).
  bool keeps = true;

  bool alloc(void** p, size_t bytes) {
    const size_t block = block_size(bytes);
    if (block >= kKeepLeast) {
      std::lock_guard<std::mutex> g(mu_);
      ++calls_;
      for (auto it = kept_.rbegin(); it != kept_.rend(); ++it)
        if (it->size == block) {
          *p = it->p;
          kept_.erase(std::next(it).base());
          kept_bytes_ -= block;
          return true;
        }
    }
    if (alloc_exact(p, block)) return true;
    if (block != bytes && dev_.alloc(p, bytes)) {
      std::lock_guard<std::mutex> g(mu_);
      unrounded_.insert(*p);
      return true;
    }
    *p = nullptr;
    return false;
  }

  // A block of exactly `bytes` from the device, to be given back to it (free).
  bool alloc_exact(void** p, size_t bytes) {
    if (dev_.alloc(p, bytes)) return true;
    peers_.drop();
    if (dev_.alloc(p, bytes)) return true;
    *p = nullptr;
    return false;
  }

  // Gives a block back to the device.
  void free(void* p) {
    if (!p) return;
    {
      std::lock_guard<std::mutex> g(mu_);
      unrounded_.erase(p);
    }
    dev_.free(p);
  }

  // Takes back a block (of `bytes` when it was allocated) that no queued or running work uses on
  // any stream: it may be handed out again at once.
  void recycle(void* p, size_t bytes) {
    if (!p) return;
    const size_t block = block_size(bytes);
    if (keeps && block >= kKeepLeast && block <= kKeepMost) {
      std::unique_lock<std::mutex> g(mu_);
      ++calls_;
      std::list<Kept> out;  // freed after the lock is given up (a free waits)
      while (kept_bytes_ + block > kKeepMost && !kept_.empty() &&
             calls_ - kept_.front().call > kStale) {
        kept_bytes_ -= kept_.front().size;
        out.splice(out.end(), kept_, kept_.begin());
      }
      const bool keep = !unrounded_.count(p) && kept_bytes_ + block <= kKeepMost;
      if (keep) {
        kept_.push_back(Kept{p, block, calls_});
        kept_bytes_ += block;
      }
      g.unlock();
      for (const Kept& k : out) dev_.free(k.p);
      if (keep) return;
    }
    free(p);
  }

  // Blocks of one released handle: they are idle once a wait has succeeded.  When it is refused
  // (another thread captures a graph, a queue has failed) queued work may still use them, and they
  // go to the device, whose free waits by itself.
  class Release {
   public:
    explicit Release(BlockPool& p) : pool_(p), idle_(p.dev_.wait()) {}
    void operator()(void* p, size_t bytes) { idle_ ? pool_.recycle(p, bytes) : pool_.free(p); }

   private:
    BlockPool& pool_;
    bool idle_;
  };

  // Frees every kept block.
  void drop() {
    std::list<Kept> out;
    {
      std::lock_guard<std::mutex> g(mu_);
      out.swap(kept_);
      kept_bytes_ = 0;
    }
    for (const Kept& k : out) dev_.free(k.p);
  }

 private:
  size_t block_size(size_t bytes) const {
    if (!keeps || bytes < kKeepLeast) return bytes;
    size_t step = kKeepLeast >> 3;
    while ((step << 4) <= bytes) step <<= 1;
    return (bytes + step - 1) / step * step;
  }

  Device dev_;
  Peers& peers_;
  std::mutex mu_;
  struct Kept {
    void* p;
    size_t size;
    unsigned call;  // when it was kept
  };
  std::list<Kept> kept_;       // oldest first; at most kKeepMost / kKeepLeast
  size_t kept_bytes_ = 0;
  unsigned calls_ = 0;
  std::set<void*> unrounded_;  // blocks smaller than their size step, never kept
};

}  // namespace bh
