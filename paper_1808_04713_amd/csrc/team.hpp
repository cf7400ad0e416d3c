// Host threads of one set-up: made as its regions need them, joined with it.  A set-up has
// a dozen parallel regions of a millisecond or less; creating their threads anew for each
// took a third of a millisecond a time.  All 16 at once took 0.5 ms, more than the whole
// analysis of a 2x2 mesh.
#pragma once
#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <exception>
#include <functional>
#include <memory>
#include <mutex>
#include <thread>
#include <vector>

namespace hdp {

class Team {
 public:
  Team() = default;
  ~Team() {
    {
      std::lock_guard<std::mutex> g(mu_);
      stop_ = true;
    }
    start_.notify_all();
    for (auto& t : threads_) t.join();
  }
  Team(const Team&) = delete;
  Team& operator=(const Team&) = delete;
  int size() const { return int(threads_.size()) + 1; }

  // f(0) .. f(n - 1), in any order, on the team and the caller; the first exception
  // is rethrown once all have ended
  void run(int n, const std::function<void(int)>& f) {
    if (n <= 0) return;
    err_ = nullptr;
    next_ = 0;
    n_ = n;
    f_ = &f;
    grow(n);
    const bool shared = n > 1 && !threads_.empty();
    if (shared) {
      {
        std::lock_guard<std::mutex> g(mu_);
        busy_ = int(threads_.size());
        ++generation_;
      }
      start_.notify_all();
    }
    take();
    if (shared) {
      std::unique_lock<std::mutex> g(mu_);
      done_.wait(g, [this] { return busy_ == 0; });
    }
    if (err_) std::rethrow_exception(err_);
  }
  // f(first, last) over ranges of 0 .. n - 1 of about `grain`
  void ranges(int64_t n, int64_t grain, const std::function<void(int64_t, int64_t)>& f) {
    const int64_t parts = (n + grain - 1) / grain;
    run(int(parts), [&](int q) { f(q * grain, std::min(n, (q + 1) * grain)); });
  }

 private:
  // threads for a region of n parts, up to one a processor and 16 in all
  void grow(int n) {
    n = std::min(n, int(std::max(1u, std::min(16u, std::thread::hardware_concurrency()))));
    try {
      threads_.reserve(size_t(n));
      while (size() < n) threads_.emplace_back([this, seen = generation_] { loop(seen); });
    } catch (const std::exception&) {   // no thread or no memory for it: fewer, down to the caller alone
    }
  }
  void take() {
    for (int q = next_++; q < n_; q = next_++) {
      try {
        (*f_)(q);
      } catch (...) {
        std::lock_guard<std::mutex> g(err_mu_);
        if (!err_) err_ = std::current_exception();
      }
    }
  }
  void loop(uint64_t seen) {   // seen: regions before this thread
    std::unique_lock<std::mutex> g(mu_);
    for (;;) {
      start_.wait(g, [&] { return stop_ || generation_ != seen; });
      if (stop_) return;
      seen = generation_;
      g.unlock();
      take();
      g.lock();
      if (--busy_ == 0) done_.notify_one();
    }
  }
  std::vector<std::thread> threads_;
  std::mutex mu_, err_mu_;
  std::condition_variable start_, done_;
  std::atomic<int> next_{0};
  int n_ = 0, busy_ = 0;
  uint64_t generation_ = 0;
  bool stop_ = false;
  const std::function<void(int)>* f_ = nullptr;
  std::exception_ptr err_;
};

// the caller's team, or one of this object's own
class TeamOr {
 public:
  explicit TeamOr(Team* t) : own_(t ? nullptr : new Team), team(t ? *t : *own_) {}

 private:
  std::unique_ptr<Team> own_;

 public:
  Team& team;
};

}  // namespace hdp
