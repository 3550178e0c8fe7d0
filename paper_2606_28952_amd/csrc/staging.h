// Pinned host staging shared by the handle-building calls.
#pragma once

#include <mutex>

#include "pbs_internal.h"

namespace pbs {

// Pinned host staging for the build's small host<->device copies, one buffer
// per device for the process's lifetime, used by one build at a time.  Copies
// through it are stream-ordered and asynchronous: an upload returns at once,
// and several downloads complete with one wait.  A copy that does not fit
// goes through pageable memory (synchronously, as before) and the buffer
// grows for the next build.
class Staging {
 public:
  explicit Staging(hipStream_t s) : s_(s) {
    int dev = 0;
    PBS_HIP(hipGetDevice(&dev));
    PBS_REQUIRE(dev >= 0 && dev < kMaxDevices, PBS_ERR_RANGE, "device index beyond the staging table");
    pool_ = &pools()[dev];
    pool_->mu.lock();
    if (!pool_->base && hipHostMalloc(&pool_->base, kInitial, hipHostMallocDefault) == hipSuccess)
      pool_->cap = kInitial;
    (void)hipGetLastError();
  }
  ~Staging() {
    // queued copies read or fill the buffer until the stream reaches them
    (void)hipStreamSynchronize(s_);
    if (wanted_ > pool_->cap) {
      if (pool_->base) (void)hipHostFree(pool_->base);
      pool_->base = nullptr;
      pool_->cap = 0;
      const size_t grown = wanted_ + wanted_ / 4;
      if (hipHostMalloc(&pool_->base, grown, hipHostMallocDefault) == hipSuccess) pool_->cap = grown;
    }
    (void)hipGetLastError();
    pool_->mu.unlock();
  }
  Staging(const Staging&) = delete;
  Staging& operator=(const Staging&) = delete;

  // memory for a slab (the handle's own, or the call's scratch arena) and its
  // uploaded parts in one copy
  void commit(Slab& b, DevBuf<char>& mem, bool temp) {
    const size_t n = b.bytes(), up = b.upload_bytes();
    if (temp)
      mem = DevBuf<char>(n, s_);
    else
      mem.alloc(n);
    b.place(mem.get());
    if (up == 0) return;
    if (void* p = take(up)) {
      b.fill_host(static_cast<char*>(p));
      PBS_HIP(hipMemcpyAsync(mem.get(), p, up, hipMemcpyHostToDevice, s_));
    } else {
      std::vector<char> image(up);
      b.fill_host(image.data());
      PBS_HIP(hipMemcpyAsync(mem.get(), image.data(), up, hipMemcpyHostToDevice, s_));
      PBS_HIP(hipStreamSynchronize(s_));  // the image ends here
    }
  }
  // n values of d into out, complete after wait()
  template <class T>
  void fetch(std::vector<T>& out, const DevBuf<T>& d, size_t n) {
    out.resize(n);
    if (!n) return;
    fetch(out.data(), d.get(), n);
  }
  template <class T>
  void fetch(T* out, const T* dev, size_t n) {
    const size_t bytes = n * sizeof(T);
    if (void* p = take(bytes)) {
      PBS_HIP(hipMemcpyAsync(p, dev, bytes, hipMemcpyDeviceToHost, s_));
      pending_.push_back({out, p, bytes});
    } else {
      PBS_HIP(hipMemcpyAsync(out, dev, bytes, hipMemcpyDeviceToHost, s_));
    }
  }
  // waits for the stream and moves the fetched values into place
  void wait() {
    PBS_HIP(hipStreamSynchronize(s_));
    for (const Pending& q : pending_) std::memcpy(q.dst, q.src, q.bytes);
    pending_.clear();
  }

 private:
  static constexpr int kMaxDevices = 64;
  static constexpr size_t kInitial = size_t(8) << 20;
  struct Pool {
    void* base = nullptr;
    size_t cap = 0;
    std::mutex mu;
  };
  struct Pending {
    void* dst;
    const void* src;
    size_t bytes;
  };
  static Pool* pools() {
    static Pool table[kMaxDevices];  // lives until the process ends
    return table;
  }
  void* take(size_t bytes) {
    const size_t need = (bytes + 255) & ~static_cast<size_t>(255);
    const size_t at = top_;
    top_ += need;
    wanted_ = std::max(wanted_, top_);
    if (!pool_->base || top_ > pool_->cap) return nullptr;
    return static_cast<char*>(pool_->base) + at;
  }
  hipStream_t s_;
  Pool* pool_ = nullptr;
  size_t top_ = 0, wanted_ = 0;
  std::vector<Pending> pending_;
};

}  // namespace pbs
