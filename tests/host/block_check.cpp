// Host-side checks of the device blocks that a pool keeps (csrc/block_cache.h) on a model of
// a device runtime: streams that are under capture or not, events that hold the point of a
// stream they were recorded at, several devices, and a limited memory that knows who may use it.
// tests/test_host_blocks.py builds and runs this.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>

#include "block_cache.h"

using spanq::BlockCache;
using spanq::DevBlock;

static int g_fail = 0;
#define CHECK(cond)                                                        \
  do {                                                                     \
    if (!(cond)) {                                                         \
      std::fprintf(stderr, "FAIL line %d: %s\n", __LINE__, #cond);         \
      ++g_fail;                                                            \
    }                                                                      \
  } while (0)

namespace {

int g_device = 0;  // the current one

struct StreamModel {
  int device = 0;
  bool captured = false;
  long issued = 0, ended = 0;             // work items enqueued, and done
  std::map<const StreamModel*, long> at;  // of each other stream: waited for its items up to here
};
struct EventModel {
  int device = 0;
  StreamModel* on = nullptr;
  long point = 0;
};
struct Memory {
  bool graph = false;  // allocated while capturing: the graph's
  int device = 0;
  size_t bytes = 0;
};

struct Model {
  using Stream = StreamModel*;
  using Event = EventModel*;
  using Error = int;
  static inline std::map<void*, Memory> memory;
  static inline std::set<EventModel*> events;
  static inline size_t limit = size_t(-1);  // bytes a device has
  struct Device {
    int before = g_device;
    explicit Device(int d) { g_device = d; }
    ~Device() { g_device = before; }
  };

  static bool capturing(Stream s) { return s->captured; }
  static Error alloc(void** p, size_t bytes, Stream s) {
    CHECK(g_device == s->device);
    size_t used = 0;
    for (const auto& m : memory) used += m.second.device == s->device ? m.second.bytes : 0;
    if (used + bytes > limit) return 2;
    *p = std::malloc(1);
    memory[*p] = Memory{s->captured, s->device, bytes};
    return 0;
  }
  static void free(void* p, Stream) {
    CHECK(memory.count(p) == 1);
    memory.erase(p);
    std::free(p);
  }
  static inline int refuse_records = 0;  // how many records fail from now on
  static Event make_event() { return *events.insert(new EventModel{g_device, nullptr, 0}).first; }
  static void destroy(Event e) {
    CHECK(events.erase(e) == 1);
    delete e;
  }
  static Error record(Event e, Stream s) {
    CHECK(events.count(e) == 1);
    if (e->device != s->device) return 1;
    if (refuse_records > 0) {
      --refuse_records;
      return 1;
    }
    e->on = s;
    e->point = s->issued;
    return 0;
  }
  static bool done(Event e) { return !e->on || e->on->ended >= e->point; }
  static Error wait(Stream s, Event e) {
    if (e->on && e->on != s) s->at[e->on] = std::max(s->at[e->on], e->point);
    return 0;
  }
};
using Cache = BlockCache<Model>;

DevBlock take(Cache& c, size_t bytes, StreamModel& s) {
  DevBlock b;
  CHECK(c.take(bytes, &s, &b) == 0);
  CHECK(b.p != nullptr && b.bytes >= bytes && Model::memory.at(b.p).bytes == b.bytes);
  ++s.issued;
  return b;
}

// A block is used again only after the work that used it before, on whatever stream.
void order() {
  Cache c(0);
  StreamModel a, b;
  DevBlock x = take(c, 1000, a);
  a.issued += 5;
  const long used = a.issued;
  c.give(x, &a);
  a.issued += 7;
  a.ended = used;
  const DevBlock y = take(c, 900, b);
  CHECK(y.p == x.p && b.at[&a] >= used);
  c.give(y, &b);
  c.clear(&a);
}

// A stream never waits for the work of another one on account of a kept block: not when it
// takes one, and not when it gives one back to a full list.
void independent_streams() {
  Cache c(0);
  StreamModel a, b;
  DevBlock x[Cache::kMaxBlocks];
  for (DevBlock& t : x) t = take(c, 70000, a);
  a.issued += 100;  // long work, not done yet
  for (const DevBlock& t : x) c.give(t, &a);
  const DevBlock y = take(c, 70000, b);
  for (const DevBlock& t : x) CHECK(y.p != t.p);
  c.give(y, &b);  // the list is full of a's blocks
  CHECK(b.at.count(&a) == 0);
  const DevBlock z = take(c, 70000, a);  // a may have its own back at any time
  bool own = false;
  for (const DevBlock& t : x) own = own || z.p == t.p;
  CHECK(own);
  c.give(z, &a);
  a.ended = a.issued;  // its work is done: b may have them, and take their places
  const DevBlock w = take(c, 70000, b), v = take(c, 1000000, b);
  own = false;
  for (const DevBlock& t : x) own = own || w.p == t.p;
  CHECK(own);
  c.give(w, &b);
  c.give(v, &b);
  const DevBlock u = take(c, 1000000, b);
  CHECK(u.p == v.p);
  c.give(u, &b);
  CHECK(Model::memory.size() == Cache::kMaxBlocks);
  c.clear(&a);
}

// At most kMaxBlocks blocks and kMaxBytes in all are kept, and no larger one.
void bounds() {
  Cache c(0);
  StreamModel s;
  const size_t half = Cache::kMaxBytes / 2;
  DevBlock x[8];
  for (int i = 0; i < 8; ++i) x[i] = take(c, i < 3 ? half : 70000, s);
  for (const DevBlock& t : x) {
    c.give(t, &s);
    size_t kept = 0, n = 0;
    for (const DevBlock& k : x)
      if (&k <= &t && Model::memory.count(k.p)) {
        kept += k.bytes;
        ++n;
      }
    CHECK(kept <= Cache::kMaxBytes && n <= Cache::kMaxBlocks && n >= 1);
  }
  const DevBlock big = take(c, Cache::kMaxBytes + 1, s);
  c.give(big, &s);
  CHECK(Model::memory.count(big.p) == 0);
  c.clear(&s);
}

// Memory allocated under capture never reaches another user, whenever it is given back;
// a stream under capture takes no kept block, and its blocks are not kept.
void capture() {
  Cache c(0);
  StreamModel a, b;
  DevBlock kept = take(c, 4096, a);
  c.give(kept, &a);
  a.captured = true;
  const DevBlock g = take(c, 4096, a), h = take(c, 4096, a);
  CHECK(g.p != kept.p && Model::memory.at(g.p).graph);
  c.give(h, &a);  // while capturing
  a.captured = false;
  c.give(g, &a);  // after the capture ended, with or without a launch
  for (int i = 0; i < 8; ++i) {
    const DevBlock t = take(c, 4096, i % 2 ? a : b);
    CHECK(!Model::memory.at(t.p).graph);
    if (i % 3) c.give(t, i % 2 ? &a : &b);
    else Model::free(t.p, nullptr);
  }
  c.clear(&a);
}

// 0 bytes (a decode step without tokens) are no block, whether or not one is kept.
void nothing() {
  Cache c(0);
  StreamModel s;
  DevBlock x;
  CHECK(c.take(0, &s, &x) == 0 && x.p == nullptr);
  c.give(take(c, 70000, s), &s);
  x = DevBlock{&c, 1, true};
  CHECK(c.take(0, &s, &x) == 0 && x.p == nullptr);
  c.give(x, &s);
  c.clear(&s);
}

// Near the memory limit an allocation passes that would pass if nothing were kept, whichever
// pool of the device keeps it; one that is too large fails, and leaves nothing in use.
void limit() {
  Cache c(0), other(0), far(1);
  StreamModel a, b, f;
  f.device = 1;
  const size_t mb = size_t{1} << 20;
  Model::limit = 100 * mb;
  c.give(take(c, 40 * mb, a), &a);
  other.give(take(other, 40 * mb, b), &b);
  const DevBlock there = take(far, 40 * mb, f);
  far.give(there, &f);
  ++b.issued;
  DevBlock x;
  CHECK(c.take(90 * mb, &a, &x) == 0 && x.p != nullptr);
  CHECK(a.at[&b] >= 1);                       // what the other pool's stream had done with its block
  CHECK(Model::memory.count(there.p) == 1);   // another device's memory is no help
  DevBlock y;
  CHECK(c.take(90 * mb, &a, &y) != 0 && y.p == nullptr);
  c.give(x, &a);
  CHECK(take(c, 90 * mb, a).p == x.p);
  c.give(x, &a);
  c.clear(&a);
  other.clear(&b);
  far.clear(&f);
  Model::limit = size_t(-1);
}

// Pools on two devices in one thread: a block is given back while the other device is the
// current one, which it still is afterwards, and is kept all the same.
void devices() {
  Cache c(1);
  StreamModel s;
  s.device = 1;
  g_device = 0;
  DevBlock x = take(c, 70000, s);
  for (int i = 0; i < 3; ++i) {
    c.give(x, &s);
    CHECK(g_device == 0);
    const DevBlock y = take(c, 70000, s);
    CHECK(y.p == x.p);
    x = y;
  }
  c.give(x, &s);
  c.clear(&s);
  CHECK(g_device == 0);
}

// An event that would not record costs one block, not the keeping of blocks from then on.
void refused_record() {
  Cache c(0);
  StreamModel s;
  DevBlock x = take(c, 70000, s);
  Model::refuse_records = 1;
  c.give(x, &s);
  CHECK(Model::memory.count(x.p) == 0);  // freed
  CHECK(Model::events.empty());          // and its event not left for the next block
  x = take(c, 70000, s);
  c.give(x, &s);
  const DevBlock y = take(c, 70000, s);
  CHECK(y.p == x.p);
  c.give(y, &s);
  c.clear(&s);
}

}  // namespace

int main() {
  order();
  independent_streams();
  bounds();
  capture();
  nothing();
  limit();
  devices();
  refused_record();
  CHECK(Model::memory.empty());
  CHECK(Model::events.empty());
  if (g_fail == 0) std::printf("all checks passed\n");
  return g_fail ? 1 : 0;
}
