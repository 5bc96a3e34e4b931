// Device blocks of destroyed plans and finished decode steps, kept for the next ones:
// freeing and allocating stream-ordered memory cost 27 and 3 us of a 75 us call.  At most
// kMaxBlocks of them and kMaxBytes in all; released with the pool.
//
// Rt is the device runtime (hip_blocks.h; tests give a model of one):
//   types Stream, Event, Error, with Error{} = success
//   type  Device: while one lives, its device is the current one (events and memory are made
//         there, and an event records only on streams of its own device)
//   bool  capturing(Stream)                     the stream is under graph capture
//   Error alloc(void**, size_t, Stream), void free(void*, Stream)    stream-ordered
//   Event make_event() (Event{} on failure), void destroy(Event)
//   Error record(Event, Stream), wait(Stream, Event)
//   bool  done(Event)                           the work it was recorded after has ended
#pragma once
#include <cstddef>
#include <mutex>
#include <vector>

namespace spanq {

// A block in use.  keep: it may be kept for another user when it is given back.  Memory
// allocated while a stream was under capture belongs to the graph (it has nothing behind it
// before the graph's first launch, and its replays reuse it), so it never is.
struct DevBlock {
  void* p = nullptr;
  size_t bytes = 0;
  bool keep = false;
};

template <class Rt>
class BlockCache {
 public:
  using Stream = typename Rt::Stream;
  using Event = typename Rt::Event;
  using Error = typename Rt::Error;
  static constexpr size_t kMaxBlocks = 4, kMaxBytes = size_t{256} << 20;

  explicit BlockCache(int device) : device_(device) {
    std::lock_guard<std::mutex> lock(all_mu_);
    next_ = first_;
    first_ = this;
  }
  ~BlockCache() {
    std::lock_guard<std::mutex> lock(all_mu_);
    BlockCache** at = &first_;
    while (*at != this) at = &(*at)->next_;
    *at = next_;
  }
  BlockCache(const BlockCache&) = delete;
  BlockCache& operator=(const BlockCache&) = delete;

  // Device memory of at least `bytes` for work on stream s: a kept block that fits without
  // much waste and that s need not wait for (given back on s, or after work that has ended),
  // else a stream-ordered allocation (always that in a stream under capture, which cannot
  // wait for an event from outside).  If that fails, what the caches of the device keep is
  // freed, this one's and other pools', and it is tried once more: keeping blocks makes no call
  // fail that passes without.  0 bytes: no block, whatever is kept.
  Error take(size_t bytes, Stream s, DevBlock* out) {
    *out = DevBlock{};
    if (bytes == 0) return Error{};
    const typename Rt::Device scope(device_);
    const bool captured = Rt::capturing(s);
    if (!captured && take_kept(bytes, s, out)) return Error{};
    const size_t got = (bytes + 0xffff) & ~static_cast<size_t>(0xffff);  // nearby sizes fit the same block later
    void* p = nullptr;
    Error e = Rt::alloc(&p, got, s);
    if (e != Error{} && !captured && free_all_kept(s)) e = Rt::alloc(&p, got, s);
    if (e == Error{}) *out = DevBlock{p, got, !captured};
    return e;
  }

  // Give a block back after the work enqueued on stream s so far (which every user of the
  // block has been ordered before): kept for the next taker, else freed on s.
  void give(const DevBlock& b, Stream s) {
    if (!b.p) return;
    const typename Rt::Device scope(device_);
    std::lock_guard<std::mutex> lock(mu_);
    Event ev{};
    if (b.keep && b.bytes <= kMaxBytes && !Rt::capturing(s)) ev = event();
    if (ev != Event{} && Rt::record(ev, s) != Error{}) {
      Rt::destroy(ev);  // (one that would not record is no use to the next block either)
      ev = Event{};
    }
    if (ev == Event{}) {
      Rt::free(b.p, s);
      return;
    }
    // Room for it: the oldest that s need not wait for go.  If that is not enough, this one
    // goes instead: no stream waits for another one's work on account of the list.
    size_t total = b.bytes;
    for (const Kept& k : kept_) total += k.bytes;
    for (auto it = kept_.begin(); (kept_.size() >= kMaxBlocks || total > kMaxBytes) && it != kept_.end();) {
      if (!free_for(*it, s)) {
        ++it;
        continue;
      }
      total -= it->bytes;
      (void)Rt::wait(s, it->done);
      Rt::free(it->p, s);
      spare_.push_back(it->done);
      it = kept_.erase(it);
    }
    if (kept_.size() >= kMaxBlocks || total > kMaxBytes) {
      Rt::free(b.p, s);
      spare_.push_back(ev);
      return;
    }
    kept_.push_back({b.p, b.bytes, ev, s});
  }

  // Free every kept block (nothing on the device uses them any more).
  void clear(Stream s) {
    const typename Rt::Device scope(device_);
    std::lock_guard<std::mutex> lock(mu_);
    for (const Kept& k : kept_) {
      Rt::free(k.p, s);
      Rt::destroy(k.done);
    }
    for (Event e : spare_) Rt::destroy(e);
    kept_.clear();
    spare_.clear();
  }

 private:
  // done: recorded, on stream `by`, after the last work that used the block; whoever takes it
  // waits for it.  (`by` is only compared: the stream may be gone, and another one in its place
  // costs a wait at most.)
  struct Kept {
    void* p;
    size_t bytes;
    Event done;
    Stream by;
  };
  static bool free_for(const Kept& k, Stream s) { return k.by == s || Rt::done(k.done); }
  bool take_kept(size_t bytes, Stream s, DevBlock* out) {
    std::lock_guard<std::mutex> lock(mu_);
    auto best = kept_.end();
    for (auto it = kept_.begin(); it != kept_.end(); ++it)
      if (it->bytes >= bytes && it->bytes <= 4 * bytes + (size_t{1} << 20) &&
          (best == kept_.end() || it->bytes < best->bytes) && free_for(*it, s))
        best = it;
    if (best == kept_.end() || Rt::wait(s, best->done) != Error{}) return false;
    *out = DevBlock{best->p, best->bytes, true};
    spare_.push_back(best->done);
    kept_.erase(best);
    return true;
  }

  // Free, on stream s, every block that a cache of this device keeps; whether there was one.
  bool free_all_kept(Stream s) {
    std::lock_guard<std::mutex> lock(all_mu_);
    bool any = false;
    for (BlockCache* c = first_; c; c = c->next_) {
      if (c->device_ != device_) continue;
      std::lock_guard<std::mutex> own(c->mu_);
      for (const Kept& k : c->kept_) {
        (void)Rt::wait(s, k.done);
        Rt::free(k.p, s);
        c->spare_.push_back(k.done);
        any = true;
      }
      c->kept_.clear();
    }
    return any;
  }

  Event event() {
    if (spare_.empty()) return Rt::make_event();
    const Event e = spare_.back();
    spare_.pop_back();
    return e;
  }
  // every cache of the process
  static inline std::mutex all_mu_;
  static inline BlockCache* first_ = nullptr;
  BlockCache* next_ = nullptr;

  int device_;
  std::mutex mu_;  // a pool is one thread's, but another pool's thread may free what this one keeps
  std::vector<Kept> kept_;
  std::vector<Event> spare_;
};

}  // namespace spanq
