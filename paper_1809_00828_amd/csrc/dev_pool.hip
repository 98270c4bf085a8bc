// Device memory of preconditioners and solver workspaces.
//
// A program that rebuilds the preconditioner of a resident problem (other
// thresholds, a parameter study) frees and allocates the same few buffers every
// time.  The driver wipes freed device memory at about 36 GB/s before it hands
// it out again, so such a loop ends up waiting for the wipe: 17 ms a build at
// elasticity 16^3 cells, p = 3 (0.6 GB of local inverses), of which 2 ms are
// work; 2.0 ms with the buffers kept (porous Poisson 48^3, p = 2: 2.9 to
// 0.86 ms).  Freed buffers are therefore kept for the next build, at most
// kPoolBytes of them in the process (the oldest go first) and only while a
// problem is alive; all are given back when the last problem is destroyed or an
// allocation of the library, of kept memory or not (dev_malloc), fails.  A kept buffer goes to its next user without the driver's
// wait, so only one that the device has done its work on is kept.  Where the wait
// for that failed, the buffer goes back to the driver, which waits itself; where
// that fails too (a capture of the calling thread forbids it), the buffer is
// parked until a later wait succeeds.
#include <hip/hip_runtime.h>

#include <deque>
#include <mutex>
#include <unordered_map>

#include "fc_internal.h"

namespace fc {
namespace {

constexpr size_t kPoolBytes = size_t(2) << 30;

struct Block {
  void* p;
  size_t bytes;
  int device;
};

struct Pool {
  std::mutex mu;
  std::unordered_map<void*, Block> out;   // handed out
  std::deque<Block> kept;                 // oldest first
  size_t kept_bytes = 0;
  std::deque<Block> parked;               // perhaps still in use, oldest first
  uint64_t parked_gone = 0;               // taken off the front of it so far
  int problems = 0;
};

// never destroyed: handles may be released by static destructors
Pool& pool() {
  static Pool* p = new Pool();
  return *p;
}

void park(Pool& P, const Block& b) {
  try {
    P.parked.push_back(b);
  } catch (const std::bad_alloc&) {   // lost rather than handed out in use
  }
}

// (hipFree waits for the device; it fails where it may not wait)
void give_back(Pool& P, const Block& b) {
  if (hipFree(b.p) != hipSuccess) {
    (void)hipGetLastError();
    park(P, b);
  }
}

void drop_oldest(Pool& P) {
  const Block b = P.kept.front();
  P.kept.pop_front();
  P.kept_bytes -= b.bytes;
  give_back(P, b);
}

void drop_all(Pool& P) {
  while (!P.kept.empty()) drop_oldest(P);
  for (size_t k = P.parked.size(); k > 0; --k) {
    const Block b = P.parked.front();
    P.parked.pop_front();
    ++P.parked_gone;
    give_back(P, b);
  }
}

// b is idle: kept for the next build, or given back.
void keep(Pool& P, const Block& b) {
  if (P.problems > 0 && b.bytes <= kPoolBytes) {
    try {
      P.kept.push_back(b);
      P.kept_bytes += b.bytes;
      while (P.kept_bytes > kPoolBytes) drop_oldest(P);
      return;
    } catch (const std::bad_alloc&) {
    }
  }
  give_back(P, b);
}

hipError_t malloc_or_drop(Pool& P, void** p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipErrorOutOfMemory && !(P.kept.empty() && P.parked.empty())) {
    (void)hipGetLastError();
    drop_all(P);
    e = hipMalloc(p, bytes);
  }
  return e;
}

}  // namespace

hipError_t dev_malloc(void** p, size_t bytes) {
  const hipError_t e = hipMalloc(p, bytes);
  if (e != hipErrorOutOfMemory) return e;
  (void)hipGetLastError();
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  return malloc_or_drop(P, p, bytes);
}

hipError_t pool_malloc(void** p, size_t bytes) {
  *p = nullptr;
  bytes = (bytes + 511) & ~size_t(511);
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  try {
    // the smallest kept buffer of this device that wastes at most a fifth
    auto best = P.kept.end();
    for (auto it = P.kept.begin(); it != P.kept.end(); ++it)
      if (it->device == dev && it->bytes >= bytes && it->bytes <= bytes + bytes / 4 &&
          (best == P.kept.end() || it->bytes < best->bytes))
        best = it;
    if (best != P.kept.end()) {
      const Block b = *best;
      P.out.emplace(b.p, b);   // first: it may throw
      P.kept.erase(best);
      P.kept_bytes -= b.bytes;
      *p = b.p;
      return hipSuccess;
    }
    P.out.reserve(P.out.size() + 1);
    e = malloc_or_drop(P, p, bytes);
    if (e == hipSuccess) P.out.emplace(*p, Block{*p, bytes, dev});
    return e;
  } catch (const std::bad_alloc&) {
    if (*p && !P.out.count(*p)) (void)hipFree(*p);
    *p = nullptr;
    return hipErrorOutOfMemory;
  }
}

void pool_free(void* p, bool idle) {
  if (!p) return;
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  auto it = P.out.find(p);
  if (it == P.out.end()) {
    (void)hipFree(p);
    return;
  }
  const Block b = it->second;
  P.out.erase(it);
  if (idle) keep(P, b);
  else give_back(P, b);
}

// hipFree waits for the whole device as hipDeviceSynchronize does, which would
// also break every graph capture in progress on any thread of the process.
hipError_t device_idle() {
  Pool& P = pool();
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  uint64_t end;   // what is parked from here on may come after the wait
  {
    std::lock_guard<std::mutex> lock(P.mu);
    end = P.parked_gone + P.parked.size();
  }
  void* p = nullptr;
  e = hipMalloc(&p, 256);
  if (e == hipSuccess) e = hipFree(p);
  std::lock_guard<std::mutex> lock(P.mu);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    if (p) park(P, Block{p, 256, dev});
    return e;
  }
  for (uint64_t k = P.parked_gone; k < end; ++k) {
    const Block b = P.parked.front();
    P.parked.pop_front();
    ++P.parked_gone;
    if (b.device == dev) keep(P, b);
    else park(P, b);
  }
  return hipSuccess;
}

hipError_t own_stream(hipStream_t* s) {
  constexpr int kDevices = 64;
  static std::mutex mu;
  static hipStream_t streams[kDevices] = {};
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!streams[dev]) {
    const hipError_t c = hipStreamCreateWithFlags(&streams[dev], hipStreamNonBlocking);
    if (c != hipSuccess) return c;
  }
  *s = streams[dev];
  return hipSuccess;
}

hipError_t copy_now(void* dst, const void* src, size_t bytes, hipMemcpyKind kind) {
  hipStream_t s;
  hipError_t e = own_stream(&s);
  if (e == hipSuccess) e = hipMemcpyAsync(dst, src, bytes, kind, s);
  return e == hipSuccess ? hipStreamSynchronize(s) : e;
}

void pool_problem_created() {
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  ++P.problems;
}

void pool_problem_destroyed() {
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  if (--P.problems == 0) drop_all(P);
}

}  // namespace fc
