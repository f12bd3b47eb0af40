// Threads of the host planners.
#pragma once

#include <algorithm>
#include <atomic>
#include <new>
#include <thread>
#include <vector>

namespace lpf {

// f(0), ..., f(n - 1) on up to `threads` threads (this one among them).
template <class F>
void parallel(int n, int threads, F &&f) {
  std::atomic<int> next(0);
  std::atomic<bool> bad(false);
  auto work = [&]() {
    try {
      for (int i; (i = next.fetch_add(1)) < n;) f(i);
    } catch (...) {
      bad = true;
    }
  };
  const int hw = std::max(1, (int)std::thread::hardware_concurrency());
  std::vector<std::thread> th;
  try {
    for (int t = 1; t < std::min({threads, n, hw}); ++t) th.emplace_back(work);
  } catch (...) {  // no more threads: the ones that run and this one do the work
  }
  work();
  for (auto &t : th) t.join();
  if (bad) throw std::bad_alloc();
}

}  // namespace lpf
