// The order of block chains on one device (host side).  Two chains that each hold a part of the
// device and need the rest end right (chain_sync.hpp), but slowly: after a wait, by the
// workgroups that happen to be there.  So chains of different streams of a process run beside each
// other only while they need no more than `room` together; a further launch waits for the chains,
// oldest first, that would be too many, and for nothing else that their streams hold: each has
// an event recorded right behind it.  Waits, launch and record are made under one lock, so
// no launch is ever between another one's look around and its entry.
// The room is counted in halves of a CU, what a tile of 8 x 8 needs.  With whole CUs, which rules
// out a meeting for certain, streams that fit together in fact wait for each other.  600 frames
// on each of several streams, s, without waits / room in halves / in whole CUs: 4 x 1080p
// fp16 4.0 / 0.83 / 0.84 (a fifth of the launches without waits met another), 1080p, 720p, 992x544
// and 832x480 together 1.22 / 0.51 / 0.59, 2 x 1080p int16 0.64 / 0.66 / 0.66, 3 x 720p 0.31 / 0.29 / 0.39.
// One entry per stream: a stream's chains follow each other, so the last one's event covers them.
// Nothing here is needed for a right result: a failed wait or record, a stream that no event can
// be recorded on (its entry has none then), or per-thread streams that share a handle cost time
// at worst.
// Ops: stream and event types, wait(stream, event), record(event &, stream) (which creates the event
// if need be), destroy(event).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <vector>

namespace nc {

template <class Ops>
class ChainGate {
 public:
  using Stream = typename Ops::Stream;
  using Event = typename Ops::Event;

  // Runs launch() (which enqueues one chain, or a graph that holds chains, that needs `share` of
  // the room, on stream) and returns what it returns; E{} is success, and a launch that failed
  // leaves no trace.
  template <class F>
  auto launch(const void* owner, Stream stream, int share, int room, F&& launch) -> decltype(launch()) {
    std::lock_guard<std::mutex> lock(m_);
    int total = share;
    bool others = false;
    for (const Entry& e : entries_)
      if (e.stream != stream) {
        total += e.share;
        others = true;
      }
    for (const Entry& e : entries_) {  // in the order of their last launches
      if (total <= room) break;
      if (e.stream == stream) continue;
      if (e.recorded) Ops::wait(stream, e.done);
      total -= e.share;
    }
    const auto err = launch();
    if (err != decltype(launch()){}) return err;
    Entry mine{stream, owner, share, false, Event{}};
    const auto it = std::find_if(entries_.begin(), entries_.end(), [&](const Entry& e) { return e.stream == stream; });
    if (it != entries_.end()) {
      // an earlier chain of the stream may still run while this one waits behind it
      mine.share = std::max(share, it->share);
      mine.done = it->done;
      entries_.erase(it);
    }
    if (others) mine.recorded = Ops::record(mine.done, stream);  // alone there is nobody to wait for it
    entries_.push_back(mine);
    return err;
  }

  // The owner's streams are idle and it goes away: entries of its launches are dropped.
  void leave(const void* owner) {
    std::lock_guard<std::mutex> lock(m_);
    for (size_t i = 0; i < entries_.size();)
      if (entries_[i].owner == owner) {
        Ops::destroy(entries_[i].done);
        entries_.erase(entries_.begin() + i);
      } else {
        ++i;
      }
  }

 private:
  struct Entry {
    Stream stream;
    const void* owner;  // of the last launch
    int share;
    bool recorded;  // done lies behind the last launch
    Event done;
  };
  std::mutex m_;
  std::vector<Entry> entries_;
};

}  // namespace nc
