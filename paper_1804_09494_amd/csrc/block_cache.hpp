// Device blocks a context has let go of and keeps for its next allocations: a
// load and partition of 2e7 elements makes 195 allocations, and hipMalloc and
// hipFree (which also waits for the device) took three quarters of its time.
// Contexts with an allocator hook or a memory limit do not use it.
#pragma once

#include <algorithm>
#include <cstddef>
#include <mutex>
#include <vector>

#include <hip/hip_runtime_api.h>

namespace tk {

// A block is handed out again while work that uses it may still be queued: the
// context orders all of its work on one stream, so that work comes first.
// Once the context has moved to another stream (stream_changed) this no longer
// holds for anything queued before: the next allocation or release waits for
// the device once, as hipFree did, and after that every kept block is idle or
// in use on the present stream only.  tk_set_stream itself does not wait: it
// may be called while a graph is captured, where a wait is an error.
//
// At most MAX_BYTES are kept (blocks above half of that never).  All of it is
// given back when the context ends, and when an allocation of any context of
// the process fails on the same device.  Only that call touches another
// context's cache, hence the lock; hipFree waits for work that still uses a block.
class BlockCache {
 public:
  static constexpr size_t MAX_BYTES = (size_t)4 << 30;
  static constexpr size_t MAX_BLOCKS = 1024;

  // room for one block more than are kept: blocks are released in destructors, which must not throw
  BlockCache() {
    blocks_.reserve(MAX_BLOCKS + 1);
    Caches& a = caches();
    std::lock_guard<std::mutex> lock(a.mu);
    a.list.push_back(this);
  }
  BlockCache(const BlockCache&) = delete;
  BlockCache& operator=(const BlockCache&) = delete;
  ~BlockCache() {
    {
      Caches& a = caches();
      std::lock_guard<std::mutex> lock(a.mu);
      a.list.erase(std::find(a.list.begin(), a.list.end(), this));
    }
    release();
  }

  void set_device(int device) { device_ = device; }

  // A block of at least `bytes` (*cap: its size), or null when the device has none.
  void* alloc(size_t bytes, size_t* cap) {
    *cap = round_up(bytes);
    void* p = settle() ? take(*cap, cap) : nullptr;
    if (p || (p = from_runtime(*cap))) return p;
    *cap = bytes;   // no more than asked for, what every context keeps given back
    if ((p = from_runtime(bytes))) return p;
    release_all(device_);
    return from_runtime(bytes);
  }

  void free(void* p, size_t cap) {
    if (cap > MAX_BYTES / 2 || !settle()) {
      (void)hipFree(p);
      return;
    }
    std::lock_guard<std::mutex> lock(mu_);
    blocks_.push_back({p, cap});
    bytes_ += cap;
    trim(MAX_BYTES, MAX_BLOCKS);
  }

  // Work queued so far is on another stream than the work to come.
  void stream_changed() { moved_ = true; }

  void release() {
    std::lock_guard<std::mutex> lock(mu_);
    trim(0, 0);
  }

 private:
  struct Block {
    void* p;
    size_t cap;
  };

  static size_t round_up(size_t n) {
    const size_t q = n < ((size_t)1 << 20) ? 4096 : (size_t)1 << 20;
    return (n + q - 1) / q * q;
  }

  struct Caches {
    std::mutex mu;
    std::vector<BlockCache*> list;
  };
  static Caches& caches() {
    static Caches* a = new Caches;   // outlives contexts that end with the process
    return *a;
  }
  static void release_all(int device) {
    Caches& a = caches();
    std::lock_guard<std::mutex> lock(a.mu);
    for (BlockCache* c : a.list)
      if (c->device_ == device) c->release();
  }

  static void* from_runtime(size_t n) {
    void* p = nullptr;
    if (hipMalloc(&p, n) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
  }

  // False when the device cannot be waited for (a capture is under way).
  bool settle() {
    if (!moved_) return true;
    int now = device_;
    (void)hipGetDevice(&now);
    if (now != device_) (void)hipSetDevice(device_);
    const bool ok = hipDeviceSynchronize() == hipSuccess;
    if (!ok) (void)hipGetLastError();
    if (now != device_) (void)hipSetDevice(now);
    if (ok) moved_ = false;
    return ok;
  }

  // the smallest block of at least `want` bytes, at most a quarter larger
  void* take(size_t want, size_t* cap) {
    std::lock_guard<std::mutex> lock(mu_);
    size_t best = blocks_.size();
    for (size_t i = 0; i < blocks_.size(); ++i)
      if (blocks_[i].cap >= want && blocks_[i].cap - want <= want / 4 + 65536 &&
          (best == blocks_.size() || blocks_[i].cap < blocks_[best].cap))
        best = i;
    if (best == blocks_.size()) return nullptr;
    void* p = blocks_[best].p;
    *cap = blocks_[best].cap;
    bytes_ -= blocks_[best].cap;
    blocks_.erase(blocks_.begin() + (std::ptrdiff_t)best);
    return p;
  }

  void trim(size_t max_bytes, size_t max_blocks) {
    size_t n = 0;
    while (n < blocks_.size() && (bytes_ > max_bytes || blocks_.size() - n > max_blocks)) {
      (void)hipFree(blocks_[n].p);
      bytes_ -= blocks_[n++].cap;
    }
    blocks_.erase(blocks_.begin(), blocks_.begin() + (std::ptrdiff_t)n);
  }

  std::mutex mu_;               // blocks_ and bytes_
  std::vector<Block> blocks_;   // oldest first
  size_t bytes_ = 0;
  int device_ = 0;
  bool moved_ = false;
};

}  // namespace tk
