// CPU checks of the device memory pool's lists (pool_core.h) over a driver that
// counts: which idle block serves a request, what is kept and for how long, a
// driver without memory, several threads. Prints "OK" on success.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <thread>
#include <vector>

#include "pool_core.h"

using grim::pool::Limits;

#define CHECK(c)                                                  \
  do {                                                            \
    if (!(c)) {                                                   \
      std::fprintf(stderr, "CHECK failed line %d: %s\n", __LINE__, #c); \
      std::exit(1);                                               \
    }                                                             \
  } while (0)

constexpr size_t MiB = size_t(1) << 20;

struct FakeDriver {
  std::mutex mu;
  std::map<void*, std::pair<size_t, int>> out;  // allocated: bytes, device
  std::map<int, size_t> used;
  size_t room = 1000 * MiB;  // per device
  size_t can_spare = ~size_t(0);
  std::atomic<double> time{0.0};
  bool watched = true;
  int allocs = 0, frees = 0;
  uintptr_t next = 4096;

  bool alloc(void** p, size_t n, int device) {
    std::lock_guard<std::mutex> lk(mu);
    if (used[device] + n > room) return false;
    *p = reinterpret_cast<void*>(next);
    next += 4096;
    out[*p] = {n, device};
    used[device] += n;
    ++allocs;
    return true;
  }
  void free(void* p, int device) {
    std::lock_guard<std::mutex> lk(mu);
    auto it = out.find(p);
    CHECK(it != out.end() && it->second.second == device);
    used[device] -= it->second.first;
    out.erase(it);
    ++frees;
  }
  double now() { return time; }
  size_t spare(int, size_t) { return can_spare; }
  bool watch() { return watched; }
};
using Pool = grim::pool::Pool<FakeDriver>;
const Limits kLimits{100 * MiB, 10.0, 2.0};

static void* get(Pool& p, size_t n, int device = 0) {
  void* b = nullptr;
  CHECK(p.alloc(&b, n, device) && b);
  return b;
}

static void test_fit() {
  FakeDriver d;
  Pool p(d, kLimits);
  CHECK(Pool::rounded(0) == 4096 && Pool::rounded(1) == 4096 && Pool::rounded(4097) == 8192);
  CHECK(Pool::rounded(MiB) == 2 * MiB && Pool::rounded(2 * MiB + 1) == 4 * MiB && Pool::rounded(MiB - 1) == MiB);
  void *a = get(p, 20 * MiB), *b = get(p, 24 * MiB), *c = get(p, 30 * MiB);
  for (void* x : {c, a, b}) p.free(x);
  CHECK(d.frees == 0 && p.idle_bytes(0) == 74 * MiB && p.idle_bytes(1) == 0 && p.idle_bytes(-1) == 74 * MiB);
  CHECK(get(p, 22 * MiB) == b);             // the smallest that fits, not the first
  void* e = get(p, 22 * MiB);               // 30 is more than a quarter larger, 20 too small
  CHECK(e != a && e != c && d.allocs == 4);
  CHECK(get(p, 25 * MiB) == c);             // 26, and 30 <= 32.5
  void* other = get(p, 20 * MiB, 1);        // blocks stay with their device
  CHECK(other != a);
  CHECK(get(p, 20 * MiB) == a);
  p.free(nullptr);
  int x;
  p.free(&x);                               // not its own: ignored
}

static void test_kept() {
  FakeDriver d;
  Pool p(d, kLimits);
  void* a = get(p, 10 * MiB);
  d.time = 2.0;                             // lived too long
  p.free(a);
  CHECK(d.frees == 1 && p.idle_bytes(0) == 0);
  p.free(get(p, 101 * MiB));                // more than may be kept
  CHECK(d.frees == 2);
  std::vector<void*> v;
  for (int i = 0; i < 6; ++i) v.push_back(get(p, 20 * MiB));
  for (int i = 0; i < 5; ++i) p.free(v[i]);
  CHECK(d.frees == 2 && p.idle_bytes(0) == 100 * MiB);
  p.free(v[5]);                             // the oldest leaves
  CHECK(d.frees == 3 && p.idle_bytes(0) == 100 * MiB && !d.out.count(v[0]));
  d.can_spare = 50 * MiB;                   // the device has grown full
  p.free(get(p, 2 * MiB));
  CHECK(p.idle_bytes(0) <= 50 * MiB && p.idle_bytes(0) >= 32 * MiB);
  d.can_spare = 0;
  p.free(get(p, 4 * MiB));
  CHECK(p.idle_bytes(0) <= 50 * MiB);
  d.can_spare = ~size_t(0);
  d.watched = false;                        // nobody would give it back
  p.free(get(p, 6 * MiB));
  CHECK(p.idle_bytes(0) == 0 && d.out.empty());
}

static void test_age() {
  FakeDriver d;
  Pool p(d, kLimits);
  CHECK(p.expire() < 0);
  void *a = get(p, 10 * MiB), *b = get(p, 20 * MiB), *c = get(p, 40 * MiB);
  p.free(a);
  d.time = 1.5;
  p.free(b);
  p.free(c);
  d.time = 9.9;
  double left = p.expire();
  CHECK(left > 0.09 && left < 0.11 && d.frees == 0);
  d.time = 10.0;
  left = p.expire();
  CHECK(left > 1.4 && left < 1.6 && d.frees == 1 && !d.out.count(a));
  void* again = get(p, 20 * MiB);           // a block in use does not age
  CHECK(again == b);
  d.time = 30.0;
  CHECK(p.expire() < 0 && d.frees == 2 && d.out.count(b) && !d.out.count(c));
  p.free(again);                            // since its last allocation: 20 s
  CHECK(d.out.empty());
  p.free(get(p, 10 * MiB));
  p.free(get(p, 10 * MiB, 1));
  p.trim(1);
  CHECK(p.idle_bytes(0) == 10 * MiB && p.idle_bytes(1) == 0);
  p.trim(-1);
  CHECK(d.out.empty() && p.expire() < 0);
}

static void test_no_memory() {
  FakeDriver d;
  Pool p(d, kLimits);
  d.room = 100 * MiB;
  void *a = get(p, 60 * MiB), *b = get(p, 20 * MiB, 1);
  p.free(a);
  p.free(b);
  void* c = get(p, 90 * MiB);               // only once the idle 60 are back
  CHECK(!d.out.count(a) && d.out.count(b) && p.idle_bytes(1) == 20 * MiB);
  void* none = &d;
  CHECK(!p.alloc(&none, 20 * MiB, 0) && none == nullptr);
  p.free(c);
  CHECK(get(p, 90 * MiB) == c);
}

// Threads that take blocks, mark them as theirs and give them back: no block is
// with two of them at a time, and every block is back with the driver at the end.
static void test_threads() {
  FakeDriver d;
  Pool p(d, kLimits);
  std::mutex mu;
  std::map<void*, int> owner;
  std::vector<std::thread> ts;
  for (int t = 0; t < 6; ++t)
    ts.emplace_back([&, t] {
      std::mt19937 rng(t);
      std::vector<void*> mine;
      for (int i = 0; i < 3000; ++i) {
        if (mine.size() < 4 && rng() % 2) {
          void* b = nullptr;
          if (!p.alloc(&b, (1 + rng() % 8) * MiB, rng() % 2)) continue;
          std::lock_guard<std::mutex> lk(mu);
          CHECK(owner.emplace(b, t).second);
          mine.push_back(b);
        } else if (!mine.empty()) {
          void* b = mine.back();
          mine.pop_back();
          {
            std::lock_guard<std::mutex> lk(mu);
            owner.erase(b);
          }
          p.free(b);
        }
        if (rng() % 50 == 0) {
          d.time = d.time + 0.5;
          (void)p.expire();
        }
        if (rng() % 500 == 0) p.trim((int)(rng() % 3) - 1);
      }
      for (void* b : mine) {
        {
          std::lock_guard<std::mutex> lk(mu);
          owner.erase(b);
        }
        p.free(b);
      }
    });
  for (auto& t : ts) t.join();
  p.trim(-1);
  CHECK(d.out.empty() && d.allocs == d.frees);
}

int main() {
  test_fit();
  test_kept();
  test_age();
  test_no_memory();
  test_threads();
  std::puts("OK");
}
