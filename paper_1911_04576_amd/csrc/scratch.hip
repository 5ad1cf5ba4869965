// Device memory of one library call.  hipMalloc is cheap, but hipFree waits
// for the device and, once a process has freed some GB, took 25 ms per GB here
// (up to 200 ms for 8 GB): a directivity call at 64 x 57 elements, 0.4 ms of
// kernels, took 16 to 18 ms with its 0.5 GB freed at the end, and took 0.37 ms
// with the block kept; macromodels of 32 types of 288 + 576 unknowns 4.31 and
// 3.94 ms.
#include <algorithm>

#include "internal.h"

namespace emsurf {
namespace {

struct Idle {
  int dev;
  void* p;
  size_t bytes;
};

std::mutex g_mu;
// least recently used first; never destroyed, so that no static destructor
// runs into a runtime that has already ended
std::vector<Idle>& idle_blocks() {
  static auto* v = new std::vector<Idle>();
  return *v;
}
int g_plans = 0;

void free_blocks(const std::vector<Idle>& blocks) {
  int dev = 0;
  if (blocks.empty() || hipGetDevice(&dev) != hipSuccess) return;
  for (const Idle& b : blocks) {
    if (b.dev != dev) (void)hipSetDevice(b.dev);
    (void)hipFree(b.p);
    if (b.dev != dev) (void)hipSetDevice(dev);
  }
}

}  // namespace

Scratch::Scratch(size_t n) {
  EMS_HIP(hipGetDevice(&dev_));
  const size_t unit = 2u << 20;
  const size_t want = std::max<size_t>(1, (n + unit - 1) / unit) * unit;
  {
    // the smallest block that holds n, of at most twice the bytes: a box
    // geometry of 2 KB would hold a workspace of GB, and the call's own
    // workspace be allocated anew
    std::lock_guard<std::mutex> lk(g_mu);
    auto& v = idle_blocks();
    auto best = v.end();
    for (auto it = v.begin(); it != v.end(); ++it)
      if (it->dev == dev_ && it->bytes >= n && it->bytes <= 2 * want && (best == v.end() || it->bytes < best->bytes))
        best = it;
    if (best != v.end()) {
      p = best->p;
      bytes = best->bytes;
      v.erase(best);
      return;
    }
  }
  device_malloc(&p, want);
  bytes = want;
}

Scratch::~Scratch() {
  // not marked idle (an error on the way): the stream may still use it, and
  // hipFree waits for the device
  if (p) (void)hipFree(p);
}

void Scratch::idle() {
  if (!p) return;
  std::vector<Idle> drop;
  if (bytes > SCRATCH_KEPT) {
    drop.push_back({dev_, p, bytes});   // (no other block would make room for it)
  } else {
    std::lock_guard<std::mutex> lk(g_mu);
    auto& v = idle_blocks();
    size_t held = bytes;
    for (const Idle& b : v)
      if (b.dev == dev_) held += b.bytes;
    for (auto it = v.begin(); it != v.end() && held > SCRATCH_KEPT;) {
      if (it->dev != dev_) { ++it; continue; }
      held -= it->bytes;
      drop.push_back(*it);
      it = v.erase(it);
    }
    v.push_back({dev_, p, bytes});
  }
  p = nullptr;
  bytes = 0;
  free_blocks(drop);
}

size_t scratch_idle_bytes() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  std::lock_guard<std::mutex> lk(g_mu);
  size_t held = 0;
  for (const Idle& b : idle_blocks())
    if (b.dev == dev) held += b.bytes;
  return held;
}

bool scratch_give_back() {
  std::vector<Idle> drop;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    drop.swap(idle_blocks());
  }
  free_blocks(drop);
  return !drop.empty();
}

void device_malloc(void** p, size_t n) {
  hipError_t e = hipMalloc(p, n);
  if (e == hipErrorOutOfMemory && scratch_give_back()) {
    (void)hipGetLastError();
    e = hipMalloc(p, n);
  }
  EMS_HIP(e);
}

void plan_opened() {
  std::lock_guard<std::mutex> lk(g_mu);
  ++g_plans;
}

void plan_closed() {
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (--g_plans > 0) return;
  }
  scratch_give_back();
}

}  // namespace emsurf

extern "C" emsurf_status emsurf_release_idle_memory(void) {
  emsurf::scratch_give_back();
  return EMSURF_OK;
}
