// kdt_blocks.h -- the blocks of device memory that the library keeps between calls.
//
// The stream-ordered pool's allocations and frees cost a call more than its kernels
// when it is small -- every free puts a marker on the stream, and after some 1500 calls
// the pool of this runtime answered in milliseconds: a build, a kNN and a count
// call over 1000 points 0.67 ms at first, 3.3 ms later; with the blocks kept
// 0.28 ms throughout.  65536 points: 1.18 and 3.3 ms, now 0.81; lists of 1000003 balls
// on 4000037 points: 7.6, now 5.6 ms.
//
// A block that goes idle may still be used by work queued on its stream.  The null stream
// lives as long as the process, so there the stream itself orders a block's next user
// after its last one.  Any other stream can be destroyed, and its handle be given to a
// new stream: what goes idle on one carries an event of that moment, and
// whoever takes the block next waits for the event in stream order, or takes it because
// the event has passed.  So nothing depends on a handle's lifetime, blocks of streams
// that are gone serve the streams that are there, and a stream may be destroyed at any time.
// The events cost a build, a kNN and a count call over 1000 points 6 us on such a stream (177 and
// 183 us; 174 on the null stream).
//
// Host code without HIP: the memory and the events come from Backend (kdt_api.hip), so
// that the rules can be run against a model of streams on any machine.
#pragma once

#include <cstddef>
#include <cstdint>
#include <iterator>
#include <list>
#include <map>
#include <memory>
#include <mutex>
#include <unordered_map>
#include <utility>

namespace kdt {

constexpr size_t kKeepBlock = size_t(128) << 20;   // the largest block kept; larger ones are
                                                   // the pool's, whose cost their work outweighs
constexpr size_t kKeepStream = size_t(512) << 20;  // idle bytes per stream
constexpr size_t kKeepAll = size_t(2) << 30;       // idle bytes in all

// Four sizes per octave, so that calls of slightly different sizes share blocks.
inline size_t block_size(size_t bytes) {
  size_t step = 256;
  while (step * 8 < bytes) step *= 2;
  return (bytes + step - 1) / step * step;
}

// Backend: types Stream and Event, and
//   bool permanent(Stream)            the stream is never destroyed
//   bool record(Event*, Stream)       a new event behind the work queued so far; false: none
//   bool passed(Event)                the event's work is done
//   bool order_after(Stream, Event)   work queued on the stream from here on waits for it
//   void forget(Event)                the event is no longer needed
//   bool free(void*, Stream)          stream-ordered
//   bool finish(Stream, const Event*) the host waits for the event (NULL: for the stream)
// Each may be called by any thread, with the lock of this class held.  No member throws:
// where host memory runs out, a block goes back to the pool instead.
template <class Backend>
class BlockCache {
 public:
  using Stream = typename Backend::Stream;

  explicit BlockCache(Backend b = Backend()) : be_(b) {}

  // An idle block of block_size(bytes) bytes for work queued on `s` from here on, or NULL.
  void* take(int dev, size_t bytes, Stream s) noexcept {
    const size_t size = block_size(bytes);
    std::lock_guard<std::mutex> lock(mu_);
    const auto at = idle_.find({dev, size});
    if (at == idle_.end()) return nullptr;
    std::list<Block>& blocks = at->second;
    for (const bool own : {true, false}) {
      for (auto it = blocks.begin(); it != blocks.end(); ++it) {
        if ((it->stream == s) != own || !usable(*it, s, own)) continue;
        void* p = it->ptr;
        if (!know(p, dev, size)) return nullptr;
        unlist(blocks, it, dev);
        return p;
      }
    }
    return nullptr;
  }

  // A block of block_size bytes, new from the pool, is in use.
  void adopt(void* p, int dev, size_t size) noexcept {
    std::lock_guard<std::mutex> lock(mu_);
    (void)know(p, dev, size);
  }

  // Blocks that only work queued on `s` so far uses.  keep: false while `s` is captured.
  void give(void* const* p, size_t n, Stream s, bool keep) noexcept {
    std::lock_guard<std::mutex> lock(mu_);
    std::shared_ptr<Mark> mark;
    bool marked = false;
    for (size_t i = 0; i < n; ++i) {
      if (!p[i]) continue;
      const auto it = live_.find(p[i]);
      if (it != live_.end()) {
        const Known b = it->second;
        live_.erase(it);
        if (keep && !marked) {
          keep = be_.permanent(s) || (mark = record(s)) != nullptr;
          marked = true;
        }
        if (keep && put(p[i], b, s, mark)) continue;
      }
      (void)be_.free(p[i], s);
    }
  }

  // The idle blocks that went idle on `s` back to the pool, in stream order; false if the
  // pool did not take one.
  bool release(int dev, Stream s) noexcept {
    std::list<Block> out;
    std::lock_guard<std::mutex> lock(mu_);
    collect(dev, &s, out);
    bool ok = true;
    for (const Block& b : out) {
      if (b.mark && !passed(*b.mark)) (void)be_.order_after(s, b.mark->event);
      ok = be_.free(b.ptr, s) && ok;
    }
    return ok;
  }

  // Every idle block of the device back to the pool, its work done, through the permanent
  // stream `s`; false if none was.
  bool release_all(int dev, Stream s) noexcept {
    std::list<Block> out;
    std::lock_guard<std::mutex> lock(mu_);
    collect(dev, nullptr, out);
    const bool any = !out.empty();
    while (!out.empty()) {
      const Block& b = out.front();
      const bool done = !b.mark || passed(*b.mark) || be_.finish(s, &b.mark->event);
      // (a block whose event cannot be waited for is left alone)
      if (done) (void)be_.free(b.ptr, s);
      out.pop_front();
    }
    return be_.finish(s, nullptr) && any;
  }

  // Idle bytes, of one stream or in all.
  size_t idle_bytes(int dev, const Stream* s) noexcept {
    std::lock_guard<std::mutex> lock(mu_);
    if (!s) return all_;
    const auto it = bytes_.find({dev, *s});
    return it == bytes_.end() ? 0 : it->second;
  }

 private:
  using Event = typename Backend::Event;
  // The event of one give(), shared by its blocks.
  struct Mark {
    Backend* be;
    Event event{};
    bool recorded = false, done = false;
    explicit Mark(Backend* b) : be(b) {}
    Mark(const Mark&) = delete;
    Mark& operator=(const Mark&) = delete;
    ~Mark() {
      if (recorded) be->forget(event);
    }
  };
  struct Block {
    void* ptr;
    size_t bytes;
    Stream stream;  // where it went idle (a name only: it may be another stream's by now)
    std::shared_ptr<Mark> mark;  // NULL: a permanent stream
    uint64_t age;
  };
  struct Known {
    int dev;
    size_t bytes;
  };
  using Lists = std::map<std::pair<int, size_t>, std::list<Block>>;

  bool know(void* p, int dev, size_t size) noexcept {
    try {
      live_[p] = Known{dev, size};
    } catch (...) {
      return false;
    }
    return true;
  }

  std::shared_ptr<Mark> record(Stream s) noexcept {
    try {
      auto m = std::make_shared<Mark>(&be_);
      m->recorded = be_.record(&m->event, s);
      if (m->recorded) return m;
    } catch (...) {
    }
    return nullptr;
  }

  bool passed(Mark& m) noexcept { return m.done || (m.done = be_.passed(m.event)); }

  // May work queued on s from here on use the block?  `own`: it went idle on s.  A block of
  // another stream is not waited for: that would tie the two streams together.
  bool usable(const Block& b, Stream s, bool own) noexcept {
    if (!b.mark) return own;
    return passed(*b.mark) || (own && be_.order_after(s, b.mark->event));
  }

  void unlist(std::list<Block>& blocks, typename std::list<Block>::iterator it, int dev) noexcept {
    uncount(dev, *it);
    blocks.erase(it);
  }
  void uncount(int dev, const Block& b) noexcept {
    all_ -= b.bytes;
    const auto at = bytes_.find({dev, b.stream});
    at->second -= b.bytes;
    if (at->second == 0) bytes_.erase(at);
  }

  // Keeps a block; false if it does not fit.
  bool put(void* p, const Known& b, Stream s, const std::shared_ptr<Mark>& mark) noexcept {
    try {
      size_t& mine = bytes_[{b.dev, s}];
      if (mine + b.bytes <= kKeepStream && make_room(b.bytes, s)) {
        idle_[{b.dev, b.bytes}].push_back(Block{p, b.bytes, s, mark, age_++});
        mine += b.bytes;
        all_ += b.bytes;
        return true;
      }
      if (mine == 0) bytes_.erase({b.dev, s});
    } catch (...) {
    }
    return false;
  }

  // Room for `bytes` more under kKeepAll: blocks of other streams whose work is done go, the
  // ones idle for longest first, so that streams that are gone do not fill the cache.
  bool make_room(size_t bytes, Stream s) noexcept {
    while (all_ + bytes > kKeepAll) {
      typename Lists::iterator list = idle_.end();
      for (auto l = idle_.begin(); l != idle_.end(); ++l)
        if (!l->second.empty() && l->second.front().mark && l->second.front().stream != s &&
            (list == idle_.end() || l->second.front().age < list->second.front().age))
          list = l;
      if (list == idle_.end() || !passed(*list->second.front().mark)) return false;
      (void)be_.free(list->second.front().ptr, s);
      unlist(list->second, list->second.begin(), list->first.first);
    }
    return true;
  }

  // Moves the idle blocks of the device (of the stream) to `out`; allocates nothing.
  void collect(int dev, const Stream* s, std::list<Block>& out) noexcept {
    for (auto& l : idle_) {
      if (l.first.first != dev) continue;
      for (auto it = l.second.begin(); it != l.second.end();) {
        const auto next = std::next(it);
        if (!s || it->stream == *s) {
          uncount(dev, *it);
          out.splice(out.end(), l.second, it);
        }
        it = next;
      }
    }
  }

  Backend be_;
  std::mutex mu_;
  Lists idle_;  // by device and size, the one idle for longest first
  std::map<std::pair<int, Stream>, size_t> bytes_;  // idle bytes by device and stream
  std::unordered_map<void*, Known> live_;           // blocks of these sizes in use
  size_t all_ = 0;
  uint64_t age_ = 0;
};

}  // namespace kdt
