// Device memory of the handles, kept between one layer's end and the next one's start.
//
// A quantisation run makes and destroys one handle per layer.  A gigabyte from hipMalloc costs
// several milliseconds, and tens where the driver has yet to clear memory freed just before: the
// whole life of 4 experts of 2048 x 7168 in eight steps took 34 to 211 ms, of which 29 were kernels.
// From kept blocks it takes 24 ms (with the present kernels).
//
// What is kept is bounded (per device, a kKeepShare-th of its memory and kBlocks blocks) and is handed
// out whole, to one handle at a time.  All of it goes back to the device when a handle ends while
// less than a kFreeShare-th of the device is free (kept blocks and the handle's own count as used),
// when an allocation of this library fails, or by gsq_release_cached().  A block comes here only
// after the device is idle, so its next user may be on any stream or thread.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

namespace gsq {

class DevicePool {
 public:
  // Of a device's memory: the most that is kept, and the least that must be free to keep any.
  static constexpr size_t kKeepShare = 16, kFreeShare = 8;
  static constexpr int kBlocks = 512;   // some 20 per handle

  // A block of at least `bytes` on the current device `dev`; *got is its size.  Kept blocks are
  // taken where they waste at most a quarter (exact sizes come back when layers repeat).
  hipError_t take(int dev, size_t bytes, void** p, size_t* got) {
    {
      std::lock_guard<std::mutex> lock(mu_);
      int best = -1;
      for (int i = 0; i < n_; ++i)
        if (b_[i].dev == dev && b_[i].bytes >= bytes && b_[i].bytes - bytes <= bytes / 4 &&
            (best < 0 || b_[i].bytes < b_[best].bytes))
          best = i;
      if (best >= 0) {
        *p = b_[best].p;
        *got = b_[best].bytes;
        remove(best);
        return hipSuccess;
      }
    }
    *got = bytes;
    return take_new(dev, bytes, p);
  }

  // A block from the runtime itself.  What is kept makes room for it, but stays where the runtime
  // refuses for another reason (a stream capture).
  hipError_t take_new(int dev, size_t bytes, void** p) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory && release(dev)) {
      (void)hipGetLastError();
      e = hipMalloc(p, bytes);
    }
    return e;
  }

  // Keep a block nothing on the device uses any more, or free it, and as many of the device's older
  // ones as bring what is kept there to `limit`.
  void give(int dev, void* p, size_t bytes, size_t limit) {
    std::lock_guard<std::mutex> lock(mu_);
    const bool keep = bytes <= limit;
    size_t kept = keep ? bytes : 0;
    for (int i = 0; i < n_; ++i) kept += b_[i].dev == dev ? b_[i].bytes : 0;
    for (int i = 0; i < n_ && kept > limit;) {   // the oldest first
      if (b_[i].dev != dev) { ++i; continue; }
      kept -= b_[i].bytes;
      (void)hipFree(b_[i].p);
      remove(i);
    }
    if (!keep) {
      (void)hipFree(p);
      return;
    }
    if (n_ == kBlocks) {
      (void)hipFree(b_[0].p);
      remove(0);
    }
    b_[n_++] = Block{p, bytes, dev};
  }

  // Free what is kept on a device (every device: -1); false if there was nothing.
  bool release(int dev) {
    std::lock_guard<std::mutex> lock(mu_);
    bool any = false;
    for (int i = 0; i < n_;) {
      if (dev >= 0 && b_[i].dev != dev) { ++i; continue; }
      (void)hipFree(b_[i].p);
      remove(i);
      any = true;
    }
    return any;
  }

  // Bytes that may be kept on the current device now: none while too little of it is free.
  static size_t limit() {
    size_t free_bytes = 0, total = 0;
    if (hipMemGetInfo(&free_bytes, &total) != hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    return free_bytes < total / kFreeShare ? 0 : total / kKeepShare;
  }

 private:
  struct Block {
    void* p;
    size_t bytes;
    int dev;
  };
  void remove(int i) {   // in order of age
    for (--n_; i < n_; ++i) b_[i] = b_[i + 1];
  }
  std::mutex mu_;
  Block b_[kBlocks] = {};
  int n_ = 0;
};

}  // namespace gsq
