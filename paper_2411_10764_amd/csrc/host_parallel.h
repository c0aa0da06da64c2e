// Loops of ensemble loading over a few host threads.  Plain C++17.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <exception>
#include <functional>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

namespace ml2 {

// The threads that the loops of one thread's scope share: started by the first
// loop that wants them, waiting between loops, joined at the scope's end
// (starting and joining them took a loop 50 us a thread).
class Team {
 public:
  Team() : outer_(std::exchange(current(), this)) {}
  ~Team() {
    current() = outer_;
    {
      std::lock_guard<std::mutex> lock(mu_);
      stop_ = true;
    }
    wake_.notify_all();
    for (std::thread &t : threads_) t.join();
  }
  Team(const Team &) = delete;
  Team &operator=(const Team &) = delete;

  // The innermost team of this thread, or nullptr.
  static Team *&current() {
    static thread_local Team *team = nullptr;
    return team;
  }

  // job() here and on up to `helpers` threads; returns when every call has.  A
  // thread that comes too late for the job does not hold it up.
  void run(int helpers, const std::function<void()> &job) {
    try {
      while ((int)threads_.size() < helpers) threads_.emplace_back([this] { loop(); });
    } catch (...) {  // no more threads, or no memory for them: fewer do the work
    }
    {
      std::lock_guard<std::mutex> lock(mu_);
      job_ = &job;
      wanted_ = helpers;
    }
    wake_.notify_all();
    job();
    std::unique_lock<std::mutex> lock(mu_);
    wanted_ = 0;
    idle_.wait(lock, [this] { return active_ == 0; });
    job_ = nullptr;
  }

 private:
  void loop() {
    std::unique_lock<std::mutex> lock(mu_);
    for (;;) {
      wake_.wait(lock, [this] { return stop_ || wanted_ > 0; });
      if (stop_) return;
      --wanted_;
      ++active_;
      const std::function<void()> *job = job_;
      lock.unlock();
      (*job)();
      lock.lock();
      if (--active_ == 0) idle_.notify_one();
    }
  }

  Team *outer_;
  std::mutex mu_;
  std::condition_variable wake_, idle_;
  std::vector<std::thread> threads_;
  const std::function<void()> *job_ = nullptr;
  int wanted_ = 0, active_ = 0;  // threads the job still takes; those in it
  bool stop_ = false;
};

// fn(i) for i in [0, n) on up to eight threads (of the current team, if there
// is one); work: the nodes handled in all, of which a thread takes 16,384 at
// least.  Fewer than 65,536 are done here: the threads' first touch of them
// costs more than it saves (loading 300 trees of depth 6, 38,100 nodes: 0.8 ms
// on two threads, 0.5 on one).  The first exception of fn is rethrown once every
// thread has ended.
template <typename Fn>
void parallel_for(int64_t n, int64_t work, Fn fn) {
  const int64_t threads = work < 65536 ? 1 : work / 16384;
  const int64_t most = std::min<int64_t>(
      {n, 8, (int64_t)std::max(1u, std::thread::hardware_concurrency()), threads});
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
  if (most < 2) {
    run();
  } else if (Team *team = std::exchange(Team::current(), nullptr)) {  // (fn's own loops stay here)
    team->run((int)most - 1, std::ref(run));
    Team::current() = team;
  } else {
    Team alone;
    alone.run((int)most - 1, std::ref(run));
  }
  if (error) std::rethrow_exception(error);
}

}  // namespace ml2
