// The pool of device memory (csrc/device_keep.h) on a device that this file plays: kCapacity bytes,
// of which `others` hold some.  Every check that fails prints a line; the exit status counts them.
#include "device_keep.h"

#include <cstdio>
#include <map>

namespace {
constexpr size_t kCapacity = size_t(1) << 30;
size_t others = 0, used = 0;
std::map<void*, size_t> blocks;
uintptr_t next_address = 1 << 20;
int failures = 0;

void check(bool ok, const char* what) {
  if (!ok) { std::printf("failed: %s\n", what); ++failures; }
}
}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t bytes) {
  if (others + used + bytes > kCapacity) return hipErrorOutOfMemory;
  *p = reinterpret_cast<void*>(next_address);
  next_address += bytes;
  blocks[*p] = bytes;
  used += bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  const auto it = blocks.find(p);
  if (it == blocks.end()) return hipErrorInvalidValue;
  used -= it->second;
  blocks.erase(it);
  return hipSuccess;
}
hipError_t hipGetDevice(int* dev) { *dev = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
}

int main() {
  constexpr size_t kMiB = size_t(1) << 20;
  spmm::DeviceKeep& keep = spmm::DeviceKeep::instance();
  auto keep_some = [&]() {   // 300 MiB idle in the pool, the device otherwise full
    others = 0;
    void* p = nullptr;
    check(keep.get(&p, 300 * kMiB) == hipSuccess, "a block to keep");
    keep.put(p, true);
    check(used == 300 * kMiB, "a block let go is kept");
    others = kCapacity - used;
  };
  // what is asked of the full device: a large and a small block of a plan, and one outside the pool
  struct { const char* what; size_t bytes; bool pooled; } asks[] = {
      {"a large block", 100 * kMiB, true}, {"a small block", size_t(4) << 10, true},
      {"a block outside the pool", 200 * kMiB, false}};
  for (const auto& ask : asks) {
    keep_some();
    void* p = nullptr;
    const hipError_t e = ask.pooled ? keep.get(&p, ask.bytes) : keep.allocate(&p, ask.bytes);
    check(e == hipSuccess && p && blocks.count(p), ask.what);
    check(used <= ask.bytes + 2 * kMiB, "the kept memory was given back");
    if (e == hipSuccess) keep.put(p, false);
    keep.give_back(-1);
    check(used == 0, "nothing is left");
    p = nullptr;
    others = kCapacity;
    check((ask.pooled ? keep.get(&p, ask.bytes) : keep.allocate(&p, ask.bytes)) == hipErrorOutOfMemory && !p,
          "with nothing to give back the error stays");
  }
  return failures;
}
