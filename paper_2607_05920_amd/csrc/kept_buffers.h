// Device buffers that contexts keep from one bootstrap to the next (host only; the device
// is a template parameter, so that the rules can be tested without one).
//
// A context keeps buffers of one size, at most kKeepMost of them, and only where eight
// times as much memory is free on the device when they come back.  They are freed with
// their context, when it asks for another size, and, every context's on the device, when
// any allocation of the library there finds no memory (alloc): what could be allocated
// without the kept buffers can be allocated with them.
#pragma once

#include <cstddef>
#include <cstdint>
#include <map>
#include <mutex>
#include <vector>

namespace fhe {

constexpr int kKeepMost = 48;
constexpr size_t kKeepFree = 8;

// Dev: int device(), the calling thread's device; status alloc(void**, size_t), status()
// on success and Dev::no_memory() where memory is short; void free(void*).
template <class Dev>
class KeptBuffers {
 public:
  using Status = typename Dev::Status;

  // Allocates on the calling thread's device.
  Status alloc(void** p, size_t bytes) {
    Status e = Dev::alloc(p, bytes);
    while (e == Dev::no_memory() && release(Dev::device())) e = Dev::alloc(p, bytes);
    return e;
  }

  // A buffer of `words` words for `owner`, a kept one if there is one; null without memory.
  uint32_t* take(const void* owner, size_t words) {
    {
      std::lock_guard<std::mutex> lg(mu_);
      auto it = kept_.find(owner);
      if (it != kept_.end()) {
        Kept& k = it->second;
        if (k.words != words) {
          drop(k);
        } else if (!k.bufs.empty()) {
          uint32_t* p = k.bufs.back();
          k.bufs.pop_back();
          return p;
        }
      }
    }
    void* p = nullptr;
    return alloc(&p, words * 4) == Status() ? (uint32_t*)p : nullptr;
  }

  // Buffers of `words` words back from `owner`, on the calling thread's device; kept unless
  // !idle (work that uses them may be queued) or more than the rules above allow.
  void give(const void* owner, const std::vector<uint32_t*>& bufs, size_t words, bool idle, size_t free_bytes) {
    std::lock_guard<std::mutex> lg(mu_);
    Kept& k = kept_[owner];
    if (k.bufs.empty()) {
      k.words = words;
      k.device = Dev::device();
    }
    for (uint32_t* p : bufs) {
      const size_t n = k.bufs.size() + 1;
      if (idle && k.words == words && n <= (size_t)kKeepMost && n * words * 4 <= free_bytes / kKeepFree)
        k.bufs.push_back(p);
      else
        Dev::free(p);
    }
  }

  // Frees what `owner` keeps.
  void forget(const void* owner) {
    std::lock_guard<std::mutex> lg(mu_);
    auto it = kept_.find(owner);
    if (it == kept_.end()) return;
    drop(it->second);
    kept_.erase(it);
  }

  // Frees every owner's buffers on `device`; whether there were any.
  bool release(int device) {
    std::lock_guard<std::mutex> lg(mu_);
    bool any = false;
    for (auto& kv : kept_) {
      if (kv.second.device != device || kv.second.bufs.empty()) continue;
      drop(kv.second);
      any = true;
    }
    return any;
  }

 private:
  struct Kept {
    std::vector<uint32_t*> bufs;
    size_t words = 0;
    int device = 0;
  };
  void drop(Kept& k) {
    for (uint32_t* p : k.bufs) Dev::free(p);
    k.bufs.clear();
  }
  std::mutex mu_;  // taken under a context's lock; takes no other
  std::map<const void*, Kept> kept_;
};

}  // namespace fhe
