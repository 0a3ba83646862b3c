// Which solver launches may be on a device at once.
//
// The workgroups of a grid wait for each other, so all of them have to be
// resident. One launch is refused when it is larger than the device
// (launch_solve); two launches from different threads could each get half of
// their workgroups in and wait until their time is up. A launch therefore takes
// its places first and gives them back when the host has waited for it. A launch
// that does not fit waits for the ones before it, in order.
#pragma once
#include <chrono>
#include <condition_variable>
#include <mutex>

namespace pdhcg {

class Places {
 public:
  // a launch of `grid` workgroups, `per` of which fit a CU
  struct Hold {
    int grid, per;
    Hold* next = nullptr;
  };

  // Waits until h and the launches that hold places are resident together in any
  // order of dispatch, but at most `limit` (a launch may also be queued behind work
  // that waits for the caller; then both go ahead, as without this).
  void take(Hold& h, int cus, std::chrono::milliseconds limit) {
    std::unique_lock<std::mutex> lock(mu_);
    append(waiting_, h);
    cv_.wait_for(lock, limit, [&] { return waiting_ == &h && fits(h, cus); });
    remove(waiting_, h);
    append(holding_, h);
    cv_.notify_all();
  }

  void give(Hold& h) {
    std::unique_lock<std::mutex> lock(mu_);
    remove(holding_, h);
    cv_.notify_all();
  }

 private:
  // Any p workgroups fit a CU, p the least of all launches' `per`: a workgroup
  // finds no room only if every CU holds p others, so up to p a CU are resident
  // whatever the order. A launch alone fits by launch_solve's own test.
  bool fits(const Hold& h, int cus) const {
    long total = h.grid;
    int p = h.per;
    for (const Hold* q = holding_; q; q = q->next) {
      total += q->grid;
      p = q->per < p ? q->per : p;
    }
    return !holding_ || total <= (long)p * cus;
  }
  static void append(Hold*& list, Hold& h) {
    Hold** at = &list;
    while (*at) at = &(*at)->next;
    h.next = nullptr;
    *at = &h;
  }
  static void remove(Hold*& list, Hold& h) {
    for (Hold** at = &list; *at; at = &(*at)->next)
      if (*at == &h) {
        *at = h.next;
        return;
      }
  }

  std::mutex mu_;
  std::condition_variable cv_;
  Hold* waiting_ = nullptr;
  Hold* holding_ = nullptr;
};

}  // namespace pdhcg
