// Device memory that plans let go, kept for the plans that follow (host code only).
#ifndef SPMM_DEVICE_KEEP_H_
#define SPMM_DEVICE_KEEP_H_

#include <hip/hip_runtime_api.h>

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

namespace spmm {

// Device memory of plans and of their construction, kept for the next plan when it is let go.
// hipMalloc and hipFree of tens of megabytes take 25 to 300 us each (they map and unmap), together
// more than building a plan of 8 M entries; a program that makes a plan per matrix, or drops and
// makes work lists, asks for the same sizes again.  Only memory that nothing uses any more comes
// here: its owner has waited for the device, or for the one stream that used it.  At most kKeepBytes
// a device are kept (0.2 % of it), each block for kKeepCalls later requests, and a block serves requests
// of two thirds of its size and more; all of it is given back when an allocation here fails, and by
// spmm_plan_destroy(NULL).  Blocks below kKeepMin go straight to the runtime, which hands those out
// without mapping.
constexpr size_t kKeepBytes = size_t(512) << 20, kKeepMin = size_t(256) << 10;
constexpr uint64_t kKeepCalls = 256;

class DeviceKeep {
 public:
  static DeviceKeep& instance() {
    static DeviceKeep* keep = new DeviceKeep();   // never destroyed: plans may outlive static data
    return *keep;
  }
  // hipMalloc; where the device has no memory left, once more with its kept blocks given back
  hipError_t allocate(void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    int dev = 0;
    if (e != hipErrorOutOfMemory || hipGetDevice(&dev) != hipSuccess) return e;
    (void)hipGetLastError();
    give_back(dev);
    return hipMalloc(p, bytes);
  }
  hipError_t get(void** p, size_t bytes) {
    if (bytes < kKeepMin) return allocate(p, bytes);
    const size_t page = bytes < (size_t(2) << 20) ? size_t(64) << 10 : size_t(2) << 20;
    bytes = (bytes + page - 1) / page * page;   // what the runtime takes for it
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (take(p, bytes, dev)) return hipSuccess;
    e = allocate(p, bytes);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mutex_);
    try { live_[*p] = Block{*p, bytes, dev, 0}; }
    catch (const std::bad_alloc&) { }             // put() then frees it
    return hipSuccess;
  }
  // idle: nothing that was enqueued still uses the block
  void put(void* p, bool idle) {
    if (!p) return;
    int dev = -1;
    if (idle && hipGetDevice(&dev) != hipSuccess) idle = false;
    {
      std::lock_guard<std::mutex> lock(mutex_);
      const auto it = live_.find(p);
      if (it != live_.end()) {
        Block b = it->second;
        live_.erase(it);
        size_t kept = b.bytes;
        for (const Block& k : kept_) kept += k.dev == b.dev ? k.bytes : 0;
        if (idle && dev == b.dev && kept <= kKeepBytes) {
          b.stamp = clock_;
          try { kept_.push_back(b); return; }
          catch (const std::bad_alloc&) { }
        }
      }
    }
    (void)hipFree(p);
  }
  void give_back(int dev /* -1: all */) {
    while (void* p = evict([&](const Block& b) { return dev < 0 || b.dev == dev; })) (void)hipFree(p);
  }

 private:
  struct Block { void* p; size_t bytes; int dev; uint64_t stamp; };

  bool take(void** p, size_t bytes, int dev) {
    bool found = false;
    uint64_t now;
    {
      std::lock_guard<std::mutex> lock(mutex_);
      now = ++clock_;
      size_t best = kept_.size();
      for (size_t i = 0; i < kept_.size(); ++i) {
        const Block& b = kept_[i];
        if (b.dev == dev && b.bytes >= bytes && b.bytes <= bytes + bytes / 2 &&
            (best == kept_.size() || b.bytes < kept_[best].bytes))
          best = i;
      }
      if (best < kept_.size()) {
        const Block b = kept_[best];
        try {
          live_[b.p] = b;
          kept_.erase(kept_.begin() + (ptrdiff_t)best);
          *p = b.p;
          found = true;
        } catch (const std::bad_alloc&) { }
      }
    }
    while (void* old = evict([&](const Block& b) { return now > b.stamp + kKeepCalls; })) (void)hipFree(old);
    return found;
  }
  template <typename Which> void* evict(Which which) {
    std::lock_guard<std::mutex> lock(mutex_);
    for (size_t i = 0; i < kept_.size(); ++i)
      if (which(kept_[i])) {
        void* p = kept_[i].p;
        kept_.erase(kept_.begin() + (ptrdiff_t)i);
        return p;
      }
    return nullptr;
  }

  std::mutex mutex_;
  std::vector<Block> kept_;
  std::unordered_map<void*, Block> live_;
  uint64_t clock_ = 0;
};

}  // namespace spmm
#endif  // SPMM_DEVICE_KEEP_H_
