// Device memory of indexes, seed tables, their workspaces and the builds'
// temporaries, kept for the next of them.
//
// hipFree hands memory to a wipe of about 40 GB/s, and hipMalloc waits for it: a
// loop over bin sizes that builds, uses and frees a 100 Mbp seed table and
// index (1.4 GB with the build's temporaries) spent 10 to 50 of its 12 to 60 ms
// a round there, against 2 ms in kernels. A block that is freed within
// kPoolShort seconds of its allocation, as in such a loop, therefore stays in a
// list per device, at most kPoolMost bytes (the 10 GB index of a q = 6 round of
// the study over bin sizes fits) and kPoolSeconds long (older ones go at the next
// call that allocates or frees); what lived longer goes back at once, and all of
// the list does when an allocation of this library fails or a server or batcher
// is about to size itself by the free memory.
//
// A block is reused by whichever thread and stream asks next, so it may only be
// given back when no work that touches it is left: pool_free is called after the
// owner's stream or the device has been waited for (hipFree waited for the
// device by itself).

#include <chrono>
#include <cstdlib>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "grim_internal.h"

namespace grim {
namespace {

constexpr size_t kPoolMost = size_t(12) << 30;
constexpr double kPoolSeconds = 10.0, kPoolShort = 2.0;

using Clock = std::chrono::steady_clock;

struct Block {
  void* p;
  size_t bytes;
  int device;
  Clock::time_point since;  // of its allocation, or since it is idle
};

struct Pool {
  std::mutex mu;
  std::unordered_map<void*, Block> live;
  std::vector<Block> idle;  // oldest first
};

// never destroyed: handles may be freed while the process ends
Pool& pool() {
  static Pool* p = new Pool;
  return *p;
}

// Takes idle blocks of the device out of the list: all, or those too old, then
// the oldest until at most `most` bytes are left.
void take_out(Pool& P, int device, bool all, size_t most, std::vector<Block>* out) {
  const auto now = Clock::now();
  size_t kept = 0;
  for (const Block& b : P.idle)
    if (b.device == device) kept += b.bytes;
  for (size_t i = 0; i < P.idle.size();) {
    const Block b = P.idle[i];
    const bool old = std::chrono::duration<double>(now - b.since).count() > kPoolSeconds;
    if (b.device == device && (all || old || kept > most)) {
      kept -= b.bytes;
      out->push_back(b);
      P.idle.erase(P.idle.begin() + (long)i);
    } else {
      ++i;
    }
  }
}

void release(const std::vector<Block>& blocks) {
  for (const Block& b : blocks) (void)hipFree(b.p);
}

hipError_t allocate(void** out, size_t bytes) {
  if (std::getenv("GRIM_POOL_TEST_FAIL")) return hipErrorOutOfMemory;  // tests: no memory for what a call still needs
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  const size_t step = bytes >= (size_t(1) << 20) ? size_t(2) << 20 : 4096;
  const size_t need = (bytes + step - 1) / step * step + (bytes == 0 ? step : 0);
  Pool& P = pool();
  std::vector<Block> old;
  {
    std::lock_guard<std::mutex> lk(P.mu);
    size_t best = P.idle.size();
    for (size_t i = 0; i < P.idle.size(); ++i) {
      const Block& b = P.idle[i];
      // the smallest that fits, but no block much larger than asked for
      if (b.device == device && b.bytes >= need && b.bytes <= need + need / 4 &&
          (best == P.idle.size() || b.bytes < P.idle[best].bytes))
        best = i;
    }
    if (best < P.idle.size()) {
      Block b = P.idle[best];
      P.idle.erase(P.idle.begin() + (long)best);
      b.since = Clock::now();
      P.live[b.p] = b;
      *out = b.p;
    }
    take_out(P, device, false, kPoolMost, &old);
  }
  release(old);
  if (*out) return hipSuccess;
  e = hipMalloc(out, need);
  if (e != hipSuccess) {
    pool_trim();
    (void)hipGetLastError();
    e = hipMalloc(out, need);
  }
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(P.mu);
  P.live[*out] = Block{*out, need, device, Clock::now()};
  return hipSuccess;
}

}  // namespace

// No exception of the lists' own memory leaves these: the C entry points call them.
hipError_t pool_alloc(void** out, size_t bytes) {
  *out = nullptr;
  hipError_t e;
  try {
    e = allocate(out, bytes);
  } catch (...) {
    if (*out) (void)hipFree(*out);
    e = hipErrorOutOfMemory;
  }
  if (e != hipSuccess) *out = nullptr;
  return e;
}

void pool_free(void* p) try {
  if (!p) return;
  Pool& P = pool();
  std::vector<Block> old;
  {
    std::lock_guard<std::mutex> lk(P.mu);
    auto it = P.live.find(p);
    if (it == P.live.end()) return;
    Block b = it->second;
    P.live.erase(it);
    const auto now = Clock::now();
    const bool brief = std::chrono::duration<double>(now - b.since).count() < kPoolShort;
    b.since = now;
    (brief ? P.idle : old).push_back(b);
    take_out(P, b.device, false, kPoolMost, &old);
  }
  release(old);
} catch (...) {
  // the block stays with the process
}

void pool_trim() try {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return;
  std::vector<Block> old;
  Pool& P = pool();
  {
    std::lock_guard<std::mutex> lk(P.mu);
    take_out(P, device, true, 0, &old);
  }
  release(old);
} catch (...) {
  // idle blocks stay for the next call
}

}  // namespace grim
