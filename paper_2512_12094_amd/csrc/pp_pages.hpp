// Host pages of output arrays, mapped before the copies into them.
#pragma once
#include <algorithm>
#include <cstddef>
#include <thread>
#include <utility>
#include <vector>

namespace pp {

// Makes every page of some arrays present and writable from a few threads, and
// leaves their contents as they are: a call that fails afterwards has not
// touched its caller's arrays.  (A page is mapped by an atomic add of zero to
// one of its bytes; the zero comes from a volatile, or the compiler would make
// it a load, which maps no writable page.)
struct Prefault {
  static constexpr size_t kMin = size_t(2) << 20;    // below: the copies fault them in
  static constexpr size_t kPage = 4096, kMaxThreads = 8;
  std::vector<std::thread> th;
  void start(const std::vector<std::pair<void*, size_t>>& parts) {
    size_t total = 0;
    for (const auto& p : parts) total += p.second;
    if (total < kMin) return;
    const size_t n = std::min<size_t>(kMaxThreads, total / (kMin / 2));
    for (size_t t = 0; t < n; ++t) {
      try {
        th.emplace_back([parts, t, n] {
          volatile unsigned char nil = 0;
          const unsigned char zero = nil;
          for (const auto& p : parts) {
            unsigned char* c = static_cast<unsigned char*>(p.first);
            const size_t lo = p.second / n * t, hi = t + 1 == n ? p.second : p.second / n * (t + 1);
            for (size_t o = lo; o < hi; o += kPage) __atomic_fetch_add(c + o, zero, __ATOMIC_RELAXED);
          }
        });
      } catch (...) {                                // no thread to be had: the copies do it
        return;
      }
    }
  }
  void join() {
    for (auto& t : th) t.join();
    th.clear();
  }
  ~Prefault() { join(); }
};

}  // namespace pp
