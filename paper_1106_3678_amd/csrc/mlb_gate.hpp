// Shares of a device among the whole-solve launches of one process (host code only).
//
// The workgroups of such a launch wait for each other, so a launch takes its share of the
// device's workgroup slots before it starts, and two of them never hold the device half
// each, waiting.  A launch that fits may pass earlier ones that do not, which keeps the
// device busy, but not more than GATE_PASSES times: then nobody who came later enters until
// the one that was passed has, so a launch that needs the whole device gets it whatever
// smaller ones keep coming.
#pragma once

#include <algorithm>
#include <condition_variable>
#include <list>
#include <mutex>

namespace mlb {

constexpr int GATE_PASSES = 16;

class ShareGate {
  struct Waiter {
    double share;
    int passed = 0;
  };
  std::mutex mu;
  std::condition_variable cv;
  std::list<Waiter> waiting;   // in order of arrival
  double used = 0;

 public:
  // Waits for a share of the device (at most 1) and takes it.
  void enter(double share) {
    std::unique_lock<std::mutex> lk(mu);
    const auto me = waiting.insert(waiting.end(), Waiter{share});
    cv.wait(lk, [&] {
      if (used + share > 1.0 + 1e-9) return false;
      return std::all_of(waiting.begin(), me, [](const Waiter& w) { return w.passed < GATE_PASSES; });
    });
    for (auto w = waiting.begin(); w != me; ++w) ++w->passed;
    waiting.erase(me);
    used += share;
    lk.unlock();
    cv.notify_all();   // whoever waited for this one to enter
  }
  void leave(double share) {
    {
      std::lock_guard<std::mutex> lk(mu);
      used = std::max(0.0, used - share);
    }
    cv.notify_all();
  }
};

}  // namespace mlb
