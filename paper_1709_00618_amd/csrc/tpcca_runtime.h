// Hooks of the context runtime used by the server (GPU library internal).
#pragma once
#include <hip/hip_runtime.h>

#include "tpcca.h"

#include <mutex>

namespace tpcca {
hipStream_t ctx_stream(tpcca_ctx_t *c);
size_t ctx_allocated(tpcca_ctx_t *c);
// Held by every call that may synchronise the device (allocation, release,
// stream and context set-up) and by graph capture, so that no capture on
// one thread meets such a call from another.
std::recursive_mutex &device_ops_lock();
// Copies queued in stream order; a copy that continues the one before it on
// both sides is joined to it (the results of a run's units lie one after the
// other, and each copy costs some 6 us).  The joined copies have to lie in one
// allocation on either side: use flush() before going to another one.
class RangeCopy {
 public:
  RangeCopy(hipMemcpyKind kind, hipStream_t stream) : kind_(kind), stream_(stream) {}
  hipError_t add(void *dst, const void *src, size_t bytes) {
    if (bytes == 0) return hipSuccess;
    hipError_t e = hipSuccess;
    if (dst != dst_ + bytes_ || src != src_ + bytes_) {
      e = flush();
      dst_ = static_cast<char *>(dst);
      src_ = static_cast<const char *>(src);
    }
    bytes_ += bytes;
    return e;
  }
  hipError_t flush() {
    const size_t n = bytes_;
    bytes_ = 0;
    return n ? hipMemcpyAsync(dst_, src_, n, kind_, stream_) : hipSuccess;
  }

 private:
  hipMemcpyKind kind_;
  hipStream_t stream_;
  char *dst_ = nullptr;
  const char *src_ = nullptr;
  size_t bytes_ = 0;
};

// The knob ranges tpcca_set_tuning accepts (n_rows bounds the row bands).
bool tuning_valid(const tpcca_tuning_t *t, int n_rows);
}  // namespace tpcca
