// The CUs of a device shared by the group-kernel launches of a process. All workgroups of such a launch wait for
// each other, one per CU: two launches of which each holds CUs that the other waits for never start. So launches
// that may run side by side must fit on the chip together; a launch that does not fit beside the unfinished ones
// of other streams is made to wait for as many of them as it takes. No HIP in here: streams and events are opaque.
#pragma once

#include <cstdint>
#include <iterator>
#include <map>
#include <vector>

namespace nmfa {

class ChipShare {
 public:
  // Workgroups are handed to the eight XCDs in turn, so a launch may need a CU more on some of them: widths are
  // counted in multiples of eight.
  static int rounded(int workgroups) { return (workgroups + 7) / 8 * 8; }

  // Forgets the launches whose event done(ev) reports complete; their events go to release(ev).
  template <class Done, class Release>
  void reap(Done done, Release release) {
    for (auto it = chains_.begin(); it != chains_.end();) {
      auto& q = it->second.q;
      size_t n = 0;
      while (n < q.size() && done(q[n].ev)) release(q[n++].ev);
      q.erase(q.begin(), q.begin() + (long)n);
      it = q.empty() ? chains_.erase(it) : std::next(it);
    }
  }

  // Other streams with unfinished launches, and the most workgroups that these can hold at once.
  int others(const void* stream, int* held) const {
    int n = 0;
    *held = 0;
    for (const auto& c : chains_)
      if (c.first != stream) ++n, *held += c.second.q.front().width;
    return n;
  }

  // Events that a launch of `width` workgroups on `stream` must wait for: the newest ones of the streams that
  // it cannot run beside, those of the longest standing first (a wait for a stream's newest event is one for all
  // of its launches), and its own stream's, whose handle may be a destroyed stream's.
  std::vector<void*> waits(const void* stream, int width, int cus) const {
    std::vector<void*> evs;
    std::vector<const Chain*> rest;
    int held = 0;
    for (const auto& c : chains_) {
      if (c.first == stream) {
        evs.push_back(c.second.q.back().ev);
      } else {
        rest.push_back(&c.second);
        held += c.second.q.front().width;
      }
    }
    while (!rest.empty() && held + width > cus) {
      size_t oldest = 0;
      for (size_t k = 1; k < rest.size(); ++k)
        if (rest[k]->newest < rest[oldest]->newest) oldest = k;
      evs.push_back(rest[oldest]->q.back().ev);
      held -= rest[oldest]->q.front().width;
      rest.erase(rest.begin() + (long)oldest);
    }
    return evs;
  }

  // A launch enqueued on `stream` behind those waits, ev recorded behind it. The launches of one stream run one
  // after the other, so only those wider than every later one count; the events of the rest go to release(ev).
  template <class Release>
  void add(const void* stream, int width, void* ev, Release release) {
    Chain& c = chains_[stream];
    while (!c.q.empty() && c.q.back().width <= width) {
      release(c.q.back().ev);
      c.q.pop_back();
    }
    c.q.push_back({width, ev});
    c.newest = ++clock_;
  }

  // Workgroups of launches that an owner has recorded into graphs: these may be replayed at any time.
  void reserve(const void* owner, int width) {
    int& w = reserved_[owner];
    w = w > width ? w : width;
  }
  void unreserve(const void* owner) { reserved_.erase(owner); }
  int reserved_by_others(const void* owner) const {
    int sum = 0;
    for (const auto& r : reserved_)
      if (r.first != owner) sum += r.second;
    return sum;
  }

 private:
  struct Launch {
    int width;
    void* ev;
  };
  struct Chain {              // unfinished launches of a stream in order; each is wider than the next
    std::vector<Launch> q;
    uint64_t newest = 0;      // when the last one was added
  };
  std::map<const void*, Chain> chains_;
  std::map<const void*, int> reserved_;
  uint64_t clock_ = 0;
};

}  // namespace nmfa
