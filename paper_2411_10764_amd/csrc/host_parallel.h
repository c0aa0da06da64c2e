// Loops of ensemble loading over a few host threads.  Plain C++17.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <exception>
#include <system_error>
#include <thread>
#include <vector>

namespace ml2 {

// fn(i) for i in [0, n) on up to eight threads; work: the nodes handled in
// all, since fewer than 32,768 are done before a thread has started.  The
// first exception of fn is rethrown once every thread has ended.
template <typename Fn>
void parallel_for(int64_t n, int64_t work, Fn fn) {
  const int64_t most = std::min<int64_t>(
      {n, 8, (int64_t)std::max(1u, std::thread::hardware_concurrency()), work / 16384});
  std::atomic<int64_t> next{0};
  std::exception_ptr error;
  std::atomic<bool> failed{false};
  auto run = [&]() {
    try {
      for (int64_t i; !failed.load(std::memory_order_relaxed) && (i = next.fetch_add(1)) < n;)
        fn(i);
    } catch (...) {
      if (!failed.exchange(true)) error = std::current_exception();
    }
  };
  std::vector<std::thread> threads;
  try {
    threads.reserve((size_t)std::max<int64_t>(most, 1));
    for (int64_t t = 1; t < most; ++t) threads.emplace_back(run);
  } catch (...) {  // no more threads, or no memory for them: fewer do the work
  }
  run();
  for (std::thread &t : threads) t.join();
  if (error) std::rethrow_exception(error);
}

}  // namespace ml2
