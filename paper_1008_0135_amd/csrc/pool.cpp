// pool.cpp -- device memory of destroyed volumes kept for the next ones.
//
// Device memory that was freed is cleared before the driver hands it out
// again, so a program that opens one cube after another waits for that
// clearing in hipMalloc: 56 of the 60 ms of opening and closing a 1 GiB cube
// with its permuted copy in a steady loop.  Blocks of destroyed volumes are
// therefore kept, at most a 1/32 of the device's memory, oldest given back
// first; all are given back when the device's last context is destroyed,
// whenever an allocation of the library fails (it is then tried again), and by
// vr_trim, for other allocators of the process.
//
// A block enters the pool only after the device was synchronised (no stream
// still uses it), so it can be handed out to work on any stream.  One lock
// guards the lists: contexts of several threads may share them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <deque>
#include <mutex>

#include "runtime.h"

namespace vr {

namespace {

struct Block {
  void* p;
  size_t bytes;
};

struct DevicePool {
  std::deque<Block> blocks;  // oldest first
  size_t total = 0, limit = 0;  // bytes held, and at most (asked for once: 6 us a question)
  int contexts = 0;
};

std::mutex g_mu;
DevicePool g_pool[kMaxDevices];

// sizes that allocations are rounded up to, so that cubes of about one size share blocks
size_t rounded(size_t bytes) {
  const size_t unit = bytes >= ((size_t)1 << 20) ? (size_t)1 << 20 : 4096;
  return (std::max<size_t>(bytes, 1) + unit - 1) / unit * unit;
}

size_t pool_limit() {
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return total_b / 32;
}

void flush_locked(DevicePool& d) {
  for (const Block& b : d.blocks) (void)hipFree(b.p);
  d.blocks.clear();
  d.total = 0;
}

int current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return -1;
  }
  return dev;
}

}  // namespace

hipError_t dev_malloc(void** p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipSuccess) return e;
  const int dev = current_device();
  if (dev < 0) return e;
  std::lock_guard<std::mutex> lk(g_mu);
  if (g_pool[dev].blocks.empty()) return e;
  (void)hipGetLastError();
  flush_locked(g_pool[dev]);
  return hipMalloc(p, bytes);
}

hipError_t dev_take(void** p, size_t bytes, size_t* got) {
  const size_t need = rounded(bytes);
  const int dev = current_device();
  if (dev >= 0) {
    std::lock_guard<std::mutex> lk(g_mu);
    DevicePool& d = g_pool[dev];
    auto best = d.blocks.end();
    for (auto it = d.blocks.begin(); it != d.blocks.end(); ++it)
      if (it->bytes >= need && it->bytes - need <= need / 8 && (best == d.blocks.end() || it->bytes < best->bytes))
        best = it;
    if (best != d.blocks.end()) {
      *p = best->p;
      *got = best->bytes;
      d.total -= best->bytes;
      d.blocks.erase(best);
      return hipSuccess;
    }
  }
  *got = need;
  return dev_malloc(p, need);
}

void dev_give(void* p, size_t bytes) {
  if (!p) return;
  const int dev = current_device();
  if (dev < 0) {
    (void)hipFree(p);
    return;
  }
  std::lock_guard<std::mutex> lk(g_mu);
  DevicePool& d = g_pool[dev];
  if (d.contexts == 0 || bytes > d.limit) {
    (void)hipFree(p);
    return;
  }
  while (!d.blocks.empty() && (d.total + bytes > d.limit || d.blocks.size() >= 64)) {
    (void)hipFree(d.blocks.front().p);
    d.total -= d.blocks.front().bytes;
    d.blocks.pop_front();
  }
  d.blocks.push_back(Block{p, bytes});
  d.total += bytes;
}

void pool_enter(int device) {
  if (device < 0 || device >= kMaxDevices) return;
  std::lock_guard<std::mutex> lk(g_mu);
  if (g_pool[device].contexts++ == 0) g_pool[device].limit = pool_limit();
}

void pool_trim(int device) {
  if (device < 0 || device >= kMaxDevices) return;
  std::lock_guard<std::mutex> lk(g_mu);
  flush_locked(g_pool[device]);
}

void pool_leave(int device) {
  if (device < 0 || device >= kMaxDevices) return;
  std::lock_guard<std::mutex> lk(g_mu);
  if (--g_pool[device].contexts == 0) flush_locked(g_pool[device]);
}

}  // namespace vr
