// Pinned host memory of the objects' read-backs.  hipHostFree waits for every
// stream of the device (288 ms beside a busy one) and is not allowed while the
// calling thread captures a stream, and hipHostMalloc takes 30 us; so a block
// goes back to a list that the next object takes it from.  The lists keep at
// most kKeep bytes; what exceeds them, and blocks larger than kMaxBlock, go back
// to the runtime.
#include <mutex>
#include <new>

#include "internal.hpp"

namespace mds {
namespace {

constexpr size_t kMinBlock = 1024, kMaxBlock = 64 * 1024, kKeep = 1 << 20;
constexpr int kClasses = 7;  // blocks of kMinBlock 2^c bytes
static_assert(kMinBlock << (kClasses - 1) == kMaxBlock, "classes");

// A free block holds the list's link.
struct FreeBlock {
  FreeBlock *next;
};
struct Pool {
  std::mutex mu;
  FreeBlock *free[kClasses] = {};
  size_t kept = 0;
};

// (constant-initialized, and nothing to destroy: an object may outlive the
// program's other statics)
Pool g_pool;

int class_of(size_t bytes) {
  int c = 0;
  while (c < kClasses && (kMinBlock << c) < bytes) ++c;
  return c;
}

}  // namespace

void *pinned_get(size_t bytes) {
  const int c = class_of(bytes);
  if (c < kClasses) {
    Pool &p = g_pool;
    std::lock_guard<std::mutex> g(p.mu);
    if (FreeBlock *b = p.free[c]) {
      p.free[c] = b->next;
      p.kept -= kMinBlock << c;
      return b;
    }
    bytes = kMinBlock << c;
  }
  void *b = nullptr;
  // (other flags would make the memory non-coherent: 1 to 2 us more a read-back)
  if (hipHostMalloc(&b, bytes, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return b;
}

void pinned_put(void *b, size_t bytes) {
  if (!b) return;
  const int c = class_of(bytes);
  if (c < kClasses) {
    Pool &p = g_pool;
    std::lock_guard<std::mutex> g(p.mu);
    if (p.kept + (kMinBlock << c) <= kKeep) {
      FreeBlock *f = new (b) FreeBlock{p.free[c]};
      p.free[c] = f;
      p.kept += kMinBlock << c;
      return;
    }
  }
  // allowed during a capture of this thread in this mode only
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  (void)hipHostFree(b);
  if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode);
}

}  // namespace mds
