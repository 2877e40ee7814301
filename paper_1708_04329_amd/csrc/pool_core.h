// The lists of the device memory pool (pool.hip): which freed blocks are kept, for
// how long, and which block serves a request. Plain C++ over a driver that
// allocates and frees, so that a CPU test can run it.
#pragma once

#include <cstddef>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace grim {
namespace pool {

struct Limits {
  size_t most;         // bytes kept per device
  double idle_s;       // seconds a block stays idle
  double brief_s;      // only blocks freed within this of their allocation are kept
};

// Driver: bool alloc(void**, size_t bytes, int device); void free(void*, int device);
//   double now(): monotonic seconds;
//   size_t spare(int device, size_t bytes): what the device's idle blocks may take up
//   now, a block of `bytes` that is about to be one of them among them;
//   bool watch(): see to it that expire() is called until it returns a negative
//   number; false where that cannot be done.
// alloc and free may be called by any thread.
template <typename Driver>
class Pool {
 public:
  Pool(Driver& d, const Limits& l) : drv(d), lim(l) {}

  // Blocks of 1 MiB and more are multiples of 2 MiB, smaller ones of 4 KiB.
  static size_t rounded(size_t bytes) {
    const size_t step = bytes >= (size_t(1) << 20) ? size_t(2) << 20 : 4096;
    return bytes == 0 ? step : (bytes + step - 1) / step * step;
  }

  // A block of at least `bytes`, idle or from the driver; where the driver has no
  // memory left, the device's idle blocks go back first.
  bool alloc(void** out, size_t bytes, int device) {
    *out = nullptr;
    const size_t need = rounded(bytes);
    {
      std::lock_guard<std::mutex> lk(mu);
      size_t best = idle.size();
      for (size_t i = 0; i < idle.size(); ++i) {
        const Block& b = idle[i];
        // the smallest that fits, but no block much larger than asked for
        if (b.device == device && b.bytes >= need && b.bytes <= need + need / 4 &&
            (best == idle.size() || b.bytes < idle[best].bytes))
          best = i;
      }
      if (best < idle.size()) {
        Block b = idle[best];
        b.since = drv.now();
        live.emplace(b.p, b);
        idle.erase(idle.begin() + (long)best);
        *out = b.p;
        return true;
      }
    }
    if (!drv.alloc(out, need, device)) {
      trim(device);
      if (!drv.alloc(out, need, device)) {
        *out = nullptr;
        return false;
      }
    }
    try {
      std::lock_guard<std::mutex> lk(mu);
      live.emplace(*out, Block{*out, need, device, drv.now()});
    } catch (...) {
      drv.free(*out, device);
      *out = nullptr;
      return false;
    }
    return true;
  }

  // Only after every use of the block on any stream is complete.
  void free(void* p) {
    if (!p) return;
    Block b;
    bool keep;
    {
      std::lock_guard<std::mutex> lk(mu);
      auto it = live.find(p);
      if (it == live.end()) return;
      b = it->second;
      live.erase(it);
      keep = drv.now() - b.since < lim.brief_s && b.bytes <= lim.most;
    }
    const size_t spare = keep ? drv.spare(b.device, b.bytes) : 0;
    keep = keep && b.bytes <= spare;
    std::vector<Block> old;
    if (keep) {
      try {
        std::lock_guard<std::mutex> lk(mu);
        b.since = drv.now();
        idle.push_back(b);
      } catch (...) {
        keep = false;
      }
    }
    if (!keep) {
      drv.free(b.p, b.device);
      return;
    }
    {
      std::lock_guard<std::mutex> lk(mu);
      size_t kept = 0;
      for (const Block& i : idle)
        if (i.device == b.device) kept += i.bytes;
      const size_t most = spare < lim.most ? spare : lim.most;
      take_out(&old, [&](const Block& i) {  // the oldest until the rest fit
        if (i.device != b.device || kept <= most) return false;
        kept -= i.bytes;
        return true;
      });
    }
    release(old);
    if (!drv.watch()) trim(b.device);
  }

  // Idle blocks of the device (-1: of all) back to the driver.
  void trim(int device) {
    std::vector<Block> old;
    {
      std::lock_guard<std::mutex> lk(mu);
      take_out(&old, [&](const Block& i) { return device < 0 || i.device == device; });
    }
    release(old);
  }

  // Blocks that have been idle for idle_s back to the driver. Returns the seconds
  // until the next one will have been, or a negative number if none is idle.
  double expire() {
    std::vector<Block> old;
    double next = -1.0;
    {
      std::lock_guard<std::mutex> lk(mu);
      const double now = drv.now();
      take_out(&old, [&](const Block& i) { return now - i.since >= lim.idle_s; });
      if (!idle.empty()) next = idle.front().since + lim.idle_s - now;
    }
    release(old);
    return next;
  }

  // Bytes idle on the device (-1: on all).
  size_t idle_bytes(int device) {
    std::lock_guard<std::mutex> lk(mu);
    size_t n = 0;
    for (const Block& i : idle) n += device < 0 || i.device == device ? i.bytes : 0;
    return n;
  }

 private:
  struct Block {
    void* p = nullptr;
    size_t bytes = 0;
    int device = 0;
    double since = 0;  // of its allocation, or since it is idle
  };

  template <typename F>
  void take_out(std::vector<Block>* out, F gone) {
    out->reserve(idle.size());
    size_t n = 0;
    for (const Block& b : idle) {
      if (gone(b)) out->push_back(b);
      else idle[n++] = b;
    }
    idle.resize(n);
  }
  void release(const std::vector<Block>& blocks) {
    for (const Block& b : blocks) drv.free(b.p, b.device);
  }

  Driver& drv;
  const Limits lim;
  std::mutex mu;
  std::unordered_map<void*, Block> live;
  std::vector<Block> idle;  // the longest idle first
};

}  // namespace pool
}  // namespace grim
