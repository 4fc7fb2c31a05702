// Which calls with image-resident launches may be under way together.  Plain C++ over a small device interface, so that it can be tested
// on the host.
//
// Such a launch needs all its work-groups on the chip at once and takes up to a CU for each, so the launches that may run at the same
// time must fit the device together.  Every call holds the CUs of its largest launch.  Calls on one stream follow each other, so a stream
// holds what its largest unfinished call does; a new call waits for other streams (largest holder first) until what is left
// and its own need fit.  Any set of calls that can overlap then fits: the newest of them was admitted with all the others counted.
// A call that is still issuing its launches has no event yet that others could wait for: a call that does not fit beside it blocks its
// host thread until it has.  All others go ahead, also while it captures and instantiates a graph.
#pragma once
#include <algorithm>
#include <condition_variable>
#include <cstddef>
#include <mutex>
#include <vector>

namespace hpf {

// Gpu: types Stream and Event; static bool finished(Event); static bool wait(Stream, Event): the stream's later work follows the event
template <class Gpu>
class Admission {
 public:
  using Stream = typename Gpu::Stream;
  using Event = typename Gpu::Event;

  // cus: CUs of the device.  Returns false when a wait could not be enqueued (the call is then not admitted).  Otherwise leave() must follow.
  bool enter(int dev, int cus, Stream s, int need) {
    std::unique_lock<std::mutex> lk(mu_);
    for (;;) {
      const Hold* own = find(dev, s);
      if (!(own && own->busy)) {   // two threads on one stream: their calls would share an entry, and the event of the first could replace that of the second
        int busy = 0, held = sum(dev, s, &busy);
        if (held + need > cus) {
          drop_finished(dev, s);
          held = sum(dev, s, &busy);
        }
        if (held + need <= cus) break;
        if (busy + need <= cus || busy == 0) {
          if (!wait_for_largest(dev, s, held + need - cus)) return false;
          break;
        }
      }
      changed_.wait(lk);
    }
    if (Hold* own = find(dev, s)) {
      own->busy = true;
      own->cus = std::max(own->cus, need);
    } else {
      holds_.push_back(Hold{dev, s, Event(), nullptr, need, false, true});
    }
    return true;
  }
  // done: recorded on s after the launches so far.  Its owner re-records it only after a later launch of its own, so waiting on it never
  // waits for too little.
  void record(int dev, Stream s, Event done, const void* owner) {
    std::lock_guard<std::mutex> lk(mu_);
    if (Hold* h = find(dev, s)) { h->ev = done; h->owner = owner; h->recorded = true; }
  }
  void leave(int dev, Stream s) {
    {
      std::lock_guard<std::mutex> lk(mu_);
      for (size_t i = 0; i < holds_.size(); ++i)
        if (holds_[i].dev == dev && holds_[i].stream == s) {
          holds_[i].busy = false;
          if (!holds_[i].recorded) holds_.erase(holds_.begin() + (std::ptrdiff_t)i);   // it failed before its first launch
          break;
        }
    }
    changed_.notify_all();
  }
  // The owner's events are about to be destroyed (device idle)
  void forget(const void* owner) {
    std::lock_guard<std::mutex> lk(mu_);
    for (size_t i = 0; i < holds_.size();) {
      Hold& h = holds_[i];
      if (h.owner == owner && !h.busy) { holds_.erase(holds_.begin() + (std::ptrdiff_t)i); continue; }
      if (h.owner == owner) { h.owner = nullptr; h.recorded = false; }   // another's call is under way on the stream
      ++i;
    }
  }

 private:
  // One per stream: its latest call, whose event covers the earlier ones.  busy: a call is between enter() and leave()
  struct Hold { int dev; Stream stream; Event ev; const void* owner; int cus; bool recorded, busy; };
  std::mutex mu_;
  std::condition_variable changed_;
  std::vector<Hold> holds_;

  Hold* find(int dev, Stream s) {
    for (Hold& h : holds_)
      if (h.dev == dev && h.stream == s) return &h;
    return nullptr;
  }
  // CUs held by other streams; *busy: of them, by calls that are still issuing
  int sum(int dev, Stream s, int* busy) const {
    int held = 0;
    *busy = 0;
    for (const Hold& h : holds_)
      if (h.dev == dev && h.stream != s) {
        held += h.cus;
        if (h.busy) *busy += h.cus;
      }
    return held;
  }
  void drop_finished(int dev, Stream s) {
    for (size_t i = 0; i < holds_.size();) {
      const Hold& h = holds_[i];
      if (h.dev == dev && h.stream != s && !h.busy && Gpu::finished(h.ev)) holds_.erase(holds_.begin() + (std::ptrdiff_t)i);
      else ++i;
    }
  }
  bool wait_for_largest(int dev, Stream s, int excess) {
    std::vector<const Hold*> others;
    for (const Hold& h : holds_)
      if (h.dev == dev && h.stream != s && !h.busy) others.push_back(&h);
    std::stable_sort(others.begin(), others.end(), [](const Hold* a, const Hold* b) { return a->cus > b->cus; });
    for (const Hold* h : others) {
      if (excess <= 0) break;
      if (!Gpu::wait(s, h->ev)) return false;
      excess -= h->cus;
    }
    return true;
  }
};

}  // namespace hpf
