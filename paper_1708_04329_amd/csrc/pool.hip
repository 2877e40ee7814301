// Device memory of indexes, seed tables, their workspaces and the builds'
// temporaries, kept for the next of them.
//
// hipFree hands memory to a wipe of about 40 GB/s, and hipMalloc waits for it: a
// loop over bin sizes that builds, uses and frees a 100 Mbp seed table and
// index (1.4 GB with the build's temporaries) spent 10 to 50 of its 12 to 60 ms
// a round there, against 2 ms in kernels. A block that is freed within
// kBrief seconds of its allocation, as in such a loop, therefore stays in a
// list per device, at most kMost bytes (the 10 GB index of a q = 6 round of
// the study over bin sizes fits) and no more than a sixteenth of the memory that
// is free; what lived longer goes back at once. A thread gives blocks back
// that have been idle for kIdle seconds, whether or not the library is called
// again; it runs only while some are. All of the list goes back when an allocation
// of this library fails, when a server or batcher is about to size itself by
// the free memory, and by grim_trim_memory.
//
// A block is reused by whichever thread and stream asks next, so it may only be
// given back when no work that touches it is left: pool_free is called after the
// owner's stream or the device has been waited for (hipFree waited for the
// device by itself).

#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <cstdlib>
#include <thread>

#include <unistd.h>

#include "grim_internal.h"
#include "pool_core.h"

namespace grim {
namespace {

constexpr size_t kMost = size_t(12) << 30;
constexpr size_t kLook = size_t(64) << 20;  // smaller blocks are kept without a look at the free memory,
constexpr double kLookAgain = 0.1;          // which a loop takes this often at most (3 us each)
constexpr double kIdle = 2.0, kBrief = 2.0;

// The thread that gives idle blocks back, and what it shares with the process's end.
struct Watch {
  std::mutex mu;
  std::condition_variable cv;
  bool running = false, stop = false;
  std::thread* thread = nullptr;
  pid_t pid = 0;  // of the process that started it: a child of fork has no such thread
};
// never destroyed, nor is the pool: handles may be freed while the process ends
Watch& watch() {
  static Watch* w = new Watch;
  return *w;
}
void watch_idle();
void end_watch() {
  Watch& w = watch();
  {
    std::lock_guard<std::mutex> lk(w.mu);
    w.stop = true;
    w.cv.notify_all();
    if (!w.thread || w.pid != getpid()) return;
  }
  w.thread->join();
}

// The device made current for a scope.
struct OnDevice {
  int before = -1, device;
  explicit OnDevice(int d) : device(d) {
    if (hipGetDevice(&before) != hipSuccess) before = device;
    if (before != device) (void)hipSetDevice(device);
  }
  ~OnDevice() {
    if (before != device) (void)hipSetDevice(before);
  }
};

struct HipDriver {
  struct Look {
    int device = -1;
    double at = 0;
    size_t spare = 0;
  };
  static constexpr size_t kDevices = 16;
  std::mutex mu;
  Look seen[kDevices];  // the last look at each device's free memory

  // Of this thread's last failed allocation: no memory, or a device in error.
  static hipError_t& failure() {
    static thread_local hipError_t e = hipErrorOutOfMemory;
    return e;
  }
  bool alloc(void** out, size_t bytes, int) {
    const hipError_t e = hipMalloc(out, bytes);
    if (e == hipSuccess) return true;
    (void)hipGetLastError();  // reported by the result alone
    failure() = e;
    return false;
  }
  void free(void* p, int device) {
    OnDevice on(device);
    (void)hipFree(p);
  }
  double now() {
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
  }
  size_t spare(int device, size_t bytes) {
    if (bytes < kLook) return kMost;
    std::lock_guard<std::mutex> lk(mu);
    Look& l = seen[(size_t)device % kDevices];
    const double t = now();
    if (l.device != device || t - l.at > kLookAgain) {
      OnDevice on(device);
      size_t fr = 0, total = 0;
      l = {device, t, hipMemGetInfo(&fr, &total) == hipSuccess ? fr / 16 : 0};
    }
    return l.spare;
  }
  bool watch() try {
    Watch& w = grim::watch();
    std::lock_guard<std::mutex> lk(w.mu);
    if (w.stop) return false;
    if (w.running) return true;
    const bool mine = w.pid == getpid();
    // its frees go through the runtime, which ends after what is registered here
    static const int at_end = std::atexit(end_watch);
    if (at_end != 0) return false;
    if (w.thread && mine) {
      w.thread->join();  // it has left its loop
      delete w.thread;
    }
    w.thread = nullptr;
    w.thread = new std::thread(watch_idle);
    w.running = true;
    w.pid = getpid();
    return true;
  } catch (...) {
    return false;
  }
};

pool::Pool<HipDriver>& blocks() {
  static auto* drv = new HipDriver;
  static auto* p = new pool::Pool<HipDriver>(*drv, pool::Limits{kMost, kIdle, kBrief});
  return *p;
}

void watch_idle() {
  Watch& w = watch();
  // its frees belong to no other thread's graph capture
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  std::unique_lock<std::mutex> lk(w.mu);
  while (!w.stop) {
    lk.unlock();
    double next = -1.0;
    try {
      next = blocks().expire();
    } catch (...) {
      next = kIdle;  // no memory for its list: later
    }
    lk.lock();
    // a block that became idle after the look sees `running` under the lock, so
    // look once more before leaving
    if (next < 0 && blocks().idle_bytes(-1) == 0) break;
    if (!w.stop) w.cv.wait_for(lk, std::chrono::duration<double>(std::max(next, 0.001)));
  }
  w.running = false;
}

}  // namespace

// No exception of the lists' own memory leaves these: the C entry points call them.
hipError_t pool_alloc(void** out, size_t bytes) {
  *out = nullptr;
  // tests: no memory for what a call still needs
  if (std::getenv("GRIM_POOL_TEST_FAIL")) return hipErrorOutOfMemory;
  int device = 0;
  const hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  try {
    HipDriver::failure() = hipErrorOutOfMemory;  // also where the lists find no host memory
    return blocks().alloc(out, bytes, device) ? hipSuccess : HipDriver::failure();
  } catch (...) {
    *out = nullptr;
    return hipErrorOutOfMemory;
  }
}

void pool_free(void* p) try {
  blocks().free(p);
} catch (...) {
  // the block stays with the process
}

void pool_trim() try {
  int device = 0;
  if (hipGetDevice(&device) == hipSuccess) blocks().trim(device);
} catch (...) {
  // idle blocks stay until the thread looks
}

}  // namespace grim

extern "C" int grim_trim_memory(void) try {
  grim::clear_error();
  grim::blocks().trim(-1);
  return GRIM_OK;
} catch (...) {
  return grim::set_error(GRIM_ENOMEM, "no host memory for the list of blocks");
}
