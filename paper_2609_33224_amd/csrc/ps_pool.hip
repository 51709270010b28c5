// Device memory of a context: buffers used again, buffers that stay, and what
// happens when the device has no more.

#include "ps_device.h"

#include <algorithm>
#include <exception>

namespace ps {

namespace {

// Every pool of the process, so that an allocation that fails can take back
// what other contexts keep idle.
struct Registry {
  std::mutex mu;
  std::vector<DevPool*> pools;
};
Registry& registry() {
  static Registry* r = new Registry;  // outlives every context
  return *r;
}

}  // namespace

DevPool::DevPool() {
  Registry& r = registry();
  std::lock_guard<std::mutex> lk(r.mu);
  r.pools.push_back(this);
}

DevPool::~DevPool() {
  {
    Registry& r = registry();
    std::lock_guard<std::mutex> lk(r.mu);
    r.pools.erase(std::remove(r.pools.begin(), r.pools.end(), this), r.pools.end());
  }
  drain();
  for (const Block& b : live_) (void)hipFree(b.p);
}

size_t DevPool::held() {
  std::lock_guard<std::mutex> lk(mu_);
  return live_bytes_ + idle_bytes_;
}

// Room for one more entry in both lists (nothing is thrown across the ABI).
bool DevPool::reserve_live() {
  try {
    if (live_.size() == live_.capacity()) live_.reserve(2 * live_.size() + 32);
    std::lock_guard<std::mutex> lk(mu_);
    const size_t need = live_.size() + 1 + idle_.size();
    if (need > idle_.capacity()) idle_.reserve(2 * need);
  } catch (const std::exception&) {
    return false;
  }
  return true;
}

hipError_t DevPool::device_alloc(void** out, size_t bytes) {
  *out = nullptr;
  if (bytes == 0) bytes = 1;
  if (!reserve_live()) return hipErrorOutOfMemory;
  // as it is; without this context's idle buffers; without any context's
  hipError_t e = hipErrorOutOfMemory;
  for (int attempt = 0; attempt < 3 && e == hipErrorOutOfMemory; ++attempt) {
    if (attempt == 1) drain();
    if (attempt == 2) {
      Registry& r = registry();
      std::lock_guard<std::mutex> lk(r.mu);
      for (DevPool* p : r.pools)
        if (p->device_ == device_) p->drain();
    }
    if (limit_ && held() + bytes > limit_) continue;
    e = hipMalloc(out, bytes);
    if (e != hipSuccess) (void)hipGetLastError();  // a later launch must not report it
  }
  if (e != hipSuccess) {
    *out = nullptr;
    return e;
  }
  live_.push_back(Block{*out, bytes});
  live_bytes_ += bytes;
  return hipSuccess;
}

hipError_t DevPool::get_block(void** out, size_t bytes) {
  *out = nullptr;
  if (bytes == 0) bytes = 1;
  if (!reserve_live()) return hipErrorOutOfMemory;
  {
    // the smallest idle buffer that fits and is at most twice as large (or
    // small anyway)
    std::lock_guard<std::mutex> lk(mu_);
    size_t best = idle_.size();
    for (size_t k = 0; k < idle_.size(); ++k)
      if (idle_[k].bytes >= bytes && idle_[k].bytes <= 2 * bytes + 65536 &&
          (best == idle_.size() || idle_[k].bytes < idle_[best].bytes))
        best = k;
    if (best < idle_.size()) {
      const Block b = idle_[best];
      idle_.erase(idle_.begin() + (long)best);
      idle_bytes_ -= b.bytes;
      live_.push_back(b);
      live_bytes_ += b.bytes;
      *out = b.p;
      return hipSuccess;
    }
  }
  return device_alloc(out, bytes);
}

void DevPool::put_idle(void* p) {
  if (!p) return;
  std::lock_guard<std::mutex> lk(mu_);
  for (size_t k = 0; k < live_.size(); ++k) {
    if (live_[k].p != p) continue;
    const Block b = live_[k];
    live_.erase(live_.begin() + (long)k);
    live_bytes_ -= b.bytes;
    idle_.push_back(b);
    idle_bytes_ += b.bytes;
    break;
  }
  while (!idle_.empty() && idle_bytes_ > std::min(kPoolIdleMax, std::max(kPoolIdleMin, 2 * live_bytes_))) {
    (void)hipFree(idle_.front().p);
    idle_bytes_ -= idle_.front().bytes;
    idle_.erase(idle_.begin());
  }
}

void DevPool::free_block(void* p) {
  if (!p) return;
  for (size_t k = 0; k < live_.size(); ++k) {
    if (live_[k].p != p) continue;
    live_bytes_ -= live_[k].bytes;
    live_.erase(live_.begin() + (long)k);
    break;
  }
  (void)hipFree(p);
}

void DevPool::drain() {
  std::lock_guard<std::mutex> lk(mu_);
  for (const Block& b : idle_) (void)hipFree(b.p);
  idle_.clear();
  idle_bytes_ = 0;
}

}  // namespace ps
