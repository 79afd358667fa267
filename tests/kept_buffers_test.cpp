// CPU test of the buffers that contexts keep between bootstraps (kept_buffers.h), on a
// stand-in device of limited memory: what could be allocated without kept buffers can be
// allocated with them, by any context; the bounds on what is kept; several threads.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <set>
#include <thread>
#include <vector>

#include "kept_buffers.h"

using namespace fhe;

static int failures = 0;
#define CHECK(c)                                                  \
  do {                                                            \
    if (!(c)) {                                                   \
      std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #c);    \
      ++failures;                                                 \
    }                                                             \
  } while (0)

// Two devices of 1000 words; an allocation takes its words from the current one.
struct FakeDevice {
  using Status = int;
  static thread_local int cur;
  static std::mutex mu;
  static size_t left[2];
  static std::map<void*, std::pair<int, size_t>> live;
  static int alloc(void** p, size_t bytes) {
    std::lock_guard<std::mutex> lg(mu);
    if (bytes / 4 > left[cur]) return 2;
    *p = std::malloc(bytes);
    left[cur] -= bytes / 4;
    live[*p] = {cur, bytes / 4};
    return 0;
  }
  static int no_memory() { return 2; }
  static void free(void* p) {
    std::lock_guard<std::mutex> lg(mu);
    auto it = live.find(p);
    CHECK(it != live.end());
    left[it->second.first] += it->second.second;
    live.erase(it);
    std::free(p);
  }
  static int device() { return cur; }
};
thread_local int FakeDevice::cur = 0;
std::mutex FakeDevice::mu;
size_t FakeDevice::left[2] = {1000, 1000};
std::map<void*, std::pair<int, size_t>> FakeDevice::live;

typedef FakeDevice D;
static const size_t kPlenty = (size_t)1 << 40;

static std::vector<uint32_t*> take_all(KeptBuffers<D>& k, const void* owner, size_t words, int n) {
  std::vector<uint32_t*> v;
  for (int i = 0; i < n; ++i) {
    v.push_back(k.take(owner, words));
    CHECK(v.back() != nullptr);
  }
  return v;
}

int main() {
  KeptBuffers<D> k;
  int a = 0, b = 0;  // two contexts
  // kept and taken again, without an allocation
  std::vector<uint32_t*> v = take_all(k, &a, 10, 20);
  k.give(&a, v, 10, true, kPlenty);
  CHECK(D::left[0] == 800);
  std::vector<uint32_t*> w = take_all(k, &a, 10, 20);
  CHECK(D::left[0] == 800 && std::set<uint32_t*>(v.begin(), v.end()) == std::set<uint32_t*>(w.begin(), w.end()));
  k.give(&a, w, 10, true, kPlenty);
  // an allocation that needs the kept memory gets it; one past the device does not
  void* p = nullptr;
  CHECK(k.alloc(&p, 900 * 4) == 0 && D::left[0] == 100);
  D::free(p);
  CHECK(D::left[0] == 1000);
  CHECK(k.alloc(&p, 1001 * 4) == 2);
  // so does another context's buffer
  k.give(&a, take_all(k, &a, 10, 48), 10, true, kPlenty);
  CHECK(D::left[0] == 520);
  uint32_t* big = k.take(&b, 700);
  CHECK(big && D::left[0] == 300);
  D::free(big);
  // buffers on another device stay
  k.give(&a, take_all(k, &a, 10, 4), 10, true, kPlenty);
  D::cur = 1;
  k.give(&b, take_all(k, &b, 10, 5), 10, true, kPlenty);
  CHECK(k.alloc(&p, 1000 * 4) == 0 && D::left[1] == 0 && D::left[0] == 960);
  D::free(p);
  D::cur = 0;
  // another size: the old ones go
  uint32_t* q = k.take(&a, 20);
  CHECK(q && D::left[0] == 980);
  k.give(&a, {q}, 20, true, kPlenty);
  // the bounds: 48 buffers, an eighth of the free memory, idle, one size
  k.forget(&a);
  CHECK(D::left[0] == 1000);
  k.give(&a, take_all(k, &a, 10, 60), 10, true, kPlenty);
  CHECK(D::left[0] == 1000 - 48 * 10);
  k.forget(&a);
  k.give(&a, take_all(k, &a, 10, 30), 10, true, 8 * 70 * 4 + 7);
  CHECK(D::left[0] == 1000 - 70);
  k.forget(&a);
  k.give(&a, take_all(k, &a, 10, 30), 10, true, 0);
  CHECK(D::left[0] == 1000);
  k.give(&a, take_all(k, &a, 10, 30), 10, false, kPlenty);
  CHECK(D::left[0] == 1000);
  v = take_all(k, &a, 10, 3);
  w = take_all(k, &a, 5, 2);
  k.give(&a, v, 10, true, kPlenty);
  k.give(&a, w, 5, true, kPlenty);  // a second size at the same time is not kept
  CHECK(D::left[0] == 970);
  k.forget(&a);
  k.forget(&b);
  CHECK(D::left[0] == 1000 && D::left[1] == 1000);
  // several threads, each with buffers of its own and allocations that take all but a tenth
  // of the device between them
  std::vector<std::thread> ts;
  for (int t = 0; t < 4; ++t)
    ts.emplace_back([&k, t] {
      int owner = t;
      for (int r = 0; r < 200; ++r) {
        std::vector<uint32_t*> u = take_all(k, &owner, 5 + t % 2, 10);
        std::set<uint32_t*> s(u.begin(), u.end());
        CHECK(s.size() == u.size());
        k.give(&owner, u, 5 + t % 2, true, kPlenty);
        void* x = nullptr;
        CHECK(k.alloc(&x, 165 * 4) == 0);
        if (x) D::free(x);
      }
      k.forget(&owner);
    });
  for (auto& t : ts) t.join();
  CHECK(D::left[0] == 1000 && D::live.empty());
  if (failures) {
    std::printf("%d FAILURES\n", failures);
    return 1;
  }
  std::printf("ALL PASSED\n");
  return 0;
}
