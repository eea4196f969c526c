// Checks of the context's block cache against a stand-in HIP runtime that
// records calls (no GPU): block_cache_check NAME exits 0 when the check holds.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>

#include "block_cache.hpp"

namespace {
std::map<void*, size_t> live;   // blocks the runtime has handed out
size_t room = (size_t)1 << 60;  // bytes it still has
int mallocs = 0, frees = 0, waits = 0;
bool capturing = false;
bool host_full = false;         // host allocations throw

void check(bool ok, const char* what) {
  if (ok) return;
  std::fprintf(stderr, "failed: %s\n", what);
  std::exit(1);
}
}  // namespace

void* operator new(size_t n) {
  if (host_full) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  ++mallocs;
  *p = nullptr;
  if (n > room) return hipErrorOutOfMemory;
  room -= n;
  *p = std::malloc(1);
  live[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  ++frees;
  check(live.count(p) == 1, "freed a block that was not handed out");
  room += live[p];
  live.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  if (capturing) return hipErrorStreamCaptureUnsupported;
  ++waits;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

using tk::BlockCache;

int main(int argc, char** argv) {
  const char* name = argc > 1 ? argv[1] : "";
  const size_t MB = (size_t)1 << 20;
  size_t cap = 0, cap2 = 0;
  if (!std::strcmp(name, "reuse")) {   // the same stream: handed out again, nothing waits
    BlockCache c;
    void* p = c.alloc(10 * MB, &cap);
    c.free(p, cap);
    check(c.alloc(9 * MB, &cap2) == p && cap2 == cap, "a block that fits is handed out again");
    check(waits == 0 && frees == 0 && mallocs == 1, "no wait, no runtime call");
    c.free(p, cap2);
  } else if (!std::strcmp(name, "stream_change")) {
    // a kept block's last work was queued on the former stream
    BlockCache c;
    void* p = c.alloc(10 * MB, &cap);
    c.free(p, cap);
    c.stream_changed();
    check(waits == 0, "changing the stream does not wait");
    check(c.alloc(10 * MB, &cap2) == p && waits == 1, "the wait comes before the block is handed out");
    c.free(p, cap2);
    check(waits == 1, "one wait per change");
    // a block released after the change was used on the former stream too
    p = c.alloc(10 * MB, &cap);
    c.stream_changed();
    c.free(p, cap);
    check(waits == 2, "the wait comes before the block is kept");
  } else if (!std::strcmp(name, "stream_change_in_capture")) {
    // no wait is possible: kept blocks stay out of use, released ones go back
    BlockCache c;
    void* p = c.alloc(10 * MB, &cap);
    c.free(p, cap);
    c.stream_changed();
    capturing = true;
    void* q = c.alloc(10 * MB, &cap2);
    check(q != p, "the block is not handed out unwaited for");
    c.free(q, cap2);
    check(frees == 1, "a released block goes back to the runtime");
    capturing = false;
    check(c.alloc(10 * MB, &cap) == p && waits == 1, "waited for once the capture is over");
    c.free(p, cap);
  } else if (!std::strcmp(name, "release_without_host_memory")) {
    // a release runs in destructors: it may not throw, and the count stays bounded
    BlockCache c;
    static void* p[1200];
    static size_t n[1200];
    for (int i = 0; i < 1200; ++i) p[i] = c.alloc(4096, &n[i]);
    // (the stand-in's own records of frees do not allocate)
    host_full = true;
    for (int i = 0; i < 1200; ++i) c.free(p[i], n[i]);
    host_full = false;
    check(live.size() == BlockCache::MAX_BLOCKS, "at most MAX_BLOCKS are kept");
  } else if (!std::strcmp(name, "other_context")) {
    // an allocation that fails gets back what the device's other contexts keep
    BlockCache a, b, far;
    far.set_device(1);
    void* p = a.alloc(10 * MB, &cap);
    void* f = far.alloc(10 * MB, &cap2);
    a.free(p, cap);
    far.free(f, cap2);
    room = 0;
    p = b.alloc(10 * MB, &cap);
    check(p != nullptr, "the other context's block was given back");
    check(frees == 1, "another device's blocks stay");
    check(b.alloc(1, &cap2) == nullptr, "nothing left: null");
    room = (size_t)1 << 60;
    b.free(p, cap);
  } else if (!std::strcmp(name, "exact_size")) {
    // sizes are rounded up; where only the size asked for is there, it is enough
    BlockCache c;
    room = 2 * MB + 1;
    void* p = c.alloc(2 * MB + 1, &cap);
    check(p && cap == 2 * MB + 1, "no more than asked for");
    c.free(p, cap);
  } else {
    std::fprintf(stderr, "no check of this name\n");
    return 2;
  }
  check(live.empty(), "everything is given back at the end");
  return 0;
}
