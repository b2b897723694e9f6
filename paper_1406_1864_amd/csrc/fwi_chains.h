// The streams and events of the launch chains beside the callers' streams.
//
// A call takes a set while it enqueues and gives it back before its work has
// run.  Another stream's call gets the set only once that work is done:
// launches behind those of a stream that is still busy, or waits for
// something, would wait too, and independent streams would queue behind each
// other.  The stream that used a set last gets it back at once, because its
// launches are in that order anyhow.  A device has at most kMaxChainSets sets;
// a call that finds all of them busy runs as one chain on its own stream.
// Sets live until the process ends (destroying streams while a process shuts
// down is not safe).
//
// Api: Stream, Event, Error types; kOk; make_stream, make_event; done(Event):
// whether what the event recorded last has run (true if nothing); shared(Stream):
// whether the handle names the same stream in every thread.
#pragma once
#include <memory>
#include <mutex>
#include <vector>

namespace fwi {

constexpr int kMaxBranches = 4;
constexpr int kMaxChainSets = 8;

template <class Api>
class ChainPool {
 public:
  using Stream = typename Api::Stream;
  using Event = typename Api::Event;
  using Error = typename Api::Error;

  struct Set {
    int device = 0;
    bool taken = false;
    Stream user{};  // the stream that used it last
    int streams = 1;  // side streams 1 .. streams - 1 exist, and their events
    bool has_fork = false;
    Stream stream[kMaxBranches] = {};
    Event fork{}, join[kMaxBranches] = {};
  };

  // A set of `device` with n - 1 side streams for a call on `user`; null
  // without an error where every set is busy.
  Error take(int device, Stream user, int n, Set** out) {
    *out = nullptr;
    Set* s = nullptr;
    {
      std::lock_guard<std::mutex> lock(mutex_);
      int count = 0;
      for (auto& c : sets_) {
        if (c->device != device) continue;
        ++count;
        if (!c->taken && c->user == user && Api::shared(user)) {
          s = c.get();
          break;
        }
      }
      if (!s)
        for (auto& c : sets_)
          if (c->device == device && !c->taken && idle(*c)) {
            s = c.get();
            break;
          }
      if (!s) {
        if (count >= kMaxChainSets) return Api::kOk;
        sets_.push_back(std::make_unique<Set>());
        s = sets_.back().get();
        s->device = device;
      }
      s->taken = true;
      s->user = user;
    }
    Error e = Api::kOk;
    if (!s->has_fork && (e = Api::make_event(&s->fork)) == Api::kOk) s->has_fork = true;
    while (e == Api::kOk && s->streams < n) {
      const int i = s->streams;
      if ((e = Api::make_event(&s->join[i])) == Api::kOk && (e = Api::make_stream(&s->stream[i])) == Api::kOk) ++s->streams;
    }
    if (e != Api::kOk) {
      give(s);
      return e;
    }
    *out = s;
    return e;
  }

  void give(Set* s) {
    std::lock_guard<std::mutex> lock(mutex_);
    s->taken = false;
  }

 private:
  static bool idle(const Set& s) {
    for (int i = 1; i < s.streams; ++i)
      if (!Api::done(s.join[i])) return false;
    return true;
  }
  std::mutex mutex_;
  std::vector<std::unique_ptr<Set>> sets_;
};

}  // namespace fwi
