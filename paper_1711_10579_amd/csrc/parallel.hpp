// Host work over independent items on a few threads.
#pragma once

#include <algorithm>
#include <atomic>
#include <exception>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

namespace pfh {

// f(0) .. f(n - 1), each once, on up to `threads` threads (the caller's among
// them; fewer when none can be started).  The first exception, after which no
// further item is begun, reaches the caller once every thread has ended.
template <typename F>
void parallel_for(int n, int threads, F f) {
  std::atomic<int> next{0};
  std::mutex mu;
  std::exception_ptr err;
  auto run = [&] {
    for (int i; (i = next.fetch_add(1)) < n;) {
      try {
        f(i);
      } catch (...) {
        std::lock_guard<std::mutex> lk(mu);
        if (!err) err = std::current_exception();
        next.store(n);
      }
    }
  };
  threads = std::min({n, threads, std::max(1, (int)std::thread::hardware_concurrency())});
  std::vector<std::thread> ts;
  if (threads > 1) {
    ts.reserve(threads - 1);
    try {
      while ((int)ts.size() < threads - 1) ts.emplace_back(run);
    } catch (const std::system_error&) {
    }
  }
  run();
  for (auto& t : ts) t.join();
  if (err) std::rethrow_exception(err);
}

}  // namespace pfh
