// Checks of the pinned metadata blocks (staging.h) on stand-ins for streams and events: every piece still holds
// what its call wrote when its reader runs, however late streams run, whether they are destroyed with work pending
// and their handles given to new ones, and whatever the sizes; plus the refusals and the events recorded.
// Usage: staging_check SEED
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <memory>
#include <random>
#include <vector>

#include "../paper_2608_11152_amd/csrc/staging.h"

namespace {

#define CHECK(c) \
  do { \
    if (!(c)) { \
      std::printf("FAILED line %d: %s\n", __LINE__, #c); \
      std::exit(1); \
    } \
  } while (0)

// A queue of work on the simulated GPU: readers of pieces, and marks of events.  It outlives its handle.
struct Queue {
  struct Op {
    const unsigned char* piece = nullptr;
    size_t n = 0;
    unsigned char want = 0;
    int event = 0;  // an event's mark, with the number of the recording
    uint64_t mark = 0;
  };
  std::deque<Op> ops;
};

struct Sim {
  std::map<int, std::shared_ptr<Queue>> handles;  // live stream handles (0: the null stream)
  std::vector<std::shared_ptr<Queue>> queues;     // every queue that may hold work
  struct Event { uint64_t recorded = 0, reached = 0; std::shared_ptr<Queue> q; };
  std::map<int, Event> events;
  int next_event = 1, device = 0, capturing = -1, bad_stream = -1;
  int records = 0, waits = 0, pinned = 0;
  int last_fail = 0;
  std::map<void*, size_t> host;
  std::vector<std::pair<const unsigned char*, size_t>> writing;

  void stream(int h) {
    handles[h] = std::make_shared<Queue>();
    queues.push_back(handles[h]);
  }
  bool step(Queue& q) {  // run the queue's next operation
    if (q.ops.empty()) return false;
    const Queue::Op op = q.ops.front();
    q.ops.pop_front();
    if (op.event) events[op.event].reached = std::max(events[op.event].reached, op.mark);
    else
      for (size_t i = 0; i < op.n; ++i) CHECK(op.piece[i] == op.want);  // (a freed block: the sanitizer's report)
    return true;
  }
};
Sim* sim;

struct SimRt {
  using Stream = int;
  using Event = int;
  static int get_device(int* d) { *d = sim->device; return 0; }
  static int is_capturing(int s, bool* c) { *c = s == sim->capturing; return 0; }
  static int event_create(int* e) { *e = sim->next_event++; sim->events[*e]; return 0; }
  static void event_destroy(int e) { sim->events.erase(e); }
  static int event_record(int e, int s) {
    if (s == sim->bad_stream) return 1;
    CHECK(sim->handles.count(s));  // the handle is alive
    auto& q = sim->handles[s];
    Sim::Event& ev = sim->events[e];
    ev.q = q;
    q->ops.push_back({nullptr, 0, 0, e, ++ev.recorded});
    ++sim->records;
    return 0;
  }
  static bool event_done(int e) { return sim->events[e].reached >= sim->events[e].recorded; }
  static int event_wait(int e) {
    ++sim->waits;
    while (!event_done(e)) CHECK(sim->step(*sim->events[e].q));
    return 0;
  }
  static int host_alloc(void** p, size_t n) { *p = std::malloc(n); sim->host[*p] = n; ++sim->pinned; return 0; }
  static void host_free(void* p) { CHECK(sim->host.erase(p)); std::free(p); }
  static const char* error_string(int) { return "error"; }
  static int hip_fail(int, const char*) { return sim->last_fail = KVP_EHIP; }
  static int fail(int code, const char*, ...) { return sim->last_fail = code; }
};
using Staging = kvp::StagingOf<SimRt>;

// A world of streams with a staging object of its own; its blocks are given back at the end.
struct World {
  Sim s;
  Staging st;
  unsigned char value = 0;
  World() { sim = &s; s.stream(0); }
  ~World() { for (auto& h : s.host) std::free(h.first); }

  void launch(int h, const Staging::Lease& l, size_t n, unsigned char v) {
    s.handles[h]->ops.push_back({static_cast<unsigned char*>(l.host), n, v, 0, 0});
  }
  int call(int h, size_t n) {  // a whole call on stream h
    Staging::Lease l;
    const int rc = st.lease(n, h, &l);
    if (rc) return rc;
    std::memset(l.host, ++value, n);
    launch(h, l, n, value);
    return st.release(l, true);
  }
  void drain() {
    for (auto& q : s.queues) while (s.step(*q)) {}
  }
};

// Calls of every size on streams that come and go, the GPU running behind at random.
void random_calls(unsigned seed, int calls) {
  World w;
  std::mt19937 rng(seed);
  auto pick = [&](int n) { return (int)(rng() % (unsigned)n); };
  const int handles = 1 + pick(6);
  for (int h = 1; h <= handles; ++h) w.s.stream(h);
  struct Held { Staging::Lease l; int h; size_t n; unsigned char v; };
  std::vector<Held> held;  // calls of other threads, between lease and release
  for (int c = 0; c < calls; ++c) {
    const int h = pick(handles + 1);
    const int kind = pick(20);
    if (kind == 0 && h > 0) {  // destroyed with its work pending; the handle goes to a new stream
      bool busy = false;
      for (const Held& x : held) busy |= x.h == h;
      if (!busy) w.s.stream(h);
      continue;
    }
    const size_t n = pick(10) == 0 ? 1 + pick(3 << 20) : 1 + pick(200 << 10);
    if (kind < 4 && held.size() < 6) {
      Held x{{}, h, n, ++w.value};
      CHECK(w.st.lease(n, h, &x.l) == KVP_OK);
      std::memset(x.l.host, x.v, n);
      held.push_back(x);
    } else if (kind < 8 && !held.empty()) {
      const Held x = held[pick((int)held.size())];
      w.launch(x.h, x.l, x.n, x.v);
      CHECK(w.st.release(x.l, true) == KVP_OK);
      for (size_t k = 0; k < held.size(); ++k)
        if (held[k].v == x.v && held[k].l.host == x.l.host) { held.erase(held.begin() + k); break; }
    } else {
      CHECK(w.call(h, n) == KVP_OK);
    }
    for (int k = pick(6); k > 0; --k) w.s.step(*w.s.queues[pick((int)w.s.queues.size())]);
  }
  for (const Held& x : held) { w.launch(x.h, x.l, x.n, x.v); CHECK(w.st.release(x.l, true) == KVP_OK); }
  w.drain();
}

// A stream destroyed with its reader pending, its handle given to a new stream that runs at once.
void recycled_handle() {
  World w;
  w.s.stream(7);
  CHECK(w.call(7, 1000) == KVP_OK);
  const auto old = w.s.handles[7];
  w.s.stream(7);
  for (int c = 0; c < 200; ++c) {
    CHECK(w.call(7, 100 << 10) == KVP_OK);
    while (w.s.step(*w.s.handles[7])) {}
  }
  while (w.s.step(*old)) {}
}

// A piece must wait for its block's event: without GPU progress the ring runs full and the host waits.
void waits_when_behind() {
  World w;
  for (int c = 0; c < 12 * 5; ++c) CHECK(w.call(0, 200 << 10) == KVP_OK);
  CHECK(w.s.waits == 0);
  CHECK(w.call(0, 200 << 10) == KVP_OK);
  CHECK(w.s.waits == 1);
  w.drain();
}

// The null stream records one event per block, also beside any number of other streams.
void events_per_block() {
  World w;
  for (int h = 1; h <= 40; ++h) {
    w.s.stream(h);
    CHECK(w.call(h, 100) == KVP_OK);
  }
  w.drain();
  const int before = w.s.records;
  CHECK(before == 40);
  for (int c = 0; c < 4096; ++c) CHECK(w.call(0, 256) == KVP_OK);  // one block of 1 MB
  CHECK(w.s.records == before);
  CHECK(w.call(0, 256) == KVP_OK);
  CHECK(w.s.records == before + 1);
  w.drain();
}

// A capturing stream is refused and takes nothing; it and the others go on afterwards.
void capture_refused() {
  World w;
  w.s.stream(3);
  CHECK(w.call(3, 100) == KVP_OK);
  w.drain();
  const int records = w.s.records;
  w.s.capturing = 3;
  for (int c = 0; c < 50; ++c) {
    Staging::Lease l;
    CHECK(w.st.lease(100, 3, &l) == KVP_EHIP && l.slot < 0);
  }
  CHECK(w.s.records == records && w.s.handles[3]->ops.empty());
  CHECK(w.call(0, 100) == KVP_OK);
  w.s.capturing = -1;
  for (int c = 0; c < 50; ++c) { CHECK(w.call(3, 100) == KVP_OK); w.drain(); }
}

// Launches that fail, on streams that take no event either, use up nothing.
void failed_launches() {
  World w;
  for (int c = 0; c < 50; ++c) {
    w.s.bad_stream = 9;
    Staging::Lease l;
    CHECK(w.st.lease(100, 9, &l) == KVP_OK);
    CHECK(w.st.release(l, false) == KVP_OK);
  }
  CHECK(w.s.pinned == 1);
  CHECK(w.call(0, 100) == KVP_OK);
  w.drain();
}

// A failed launch does not give back a block of the null stream whose event cannot be recorded: calls before it may
// still be reading their pieces.
void failed_launch_in_a_shared_block() {
  World w;
  w.s.stream(5);
  CHECK(w.call(0, 100 << 10) == KVP_OK);
  Staging::Lease a, b;
  CHECK(w.st.lease(100, 0, &a) == KVP_OK);
  CHECK(w.st.lease(1 << 20, 0, &b) == KVP_OK);  // no room: the block closes with the call that holds a
  w.s.bad_stream = 0;
  (void)w.st.release(a, false);
  w.s.bad_stream = -1;
  for (int c = 0; c < 50; ++c) {
    CHECK(w.call(5, 100 << 10) == KVP_OK);
    while (w.s.step(*w.s.handles[5])) {}
  }
  CHECK(w.st.release(b, true) == KVP_OK);
  w.drain();
}

// Eight calls at once on other streams beside the null stream's block of each of four devices; the thirteenth
// block is refused.
void concurrent_calls() {
  World w;
  for (int d = 0; d < 4; ++d) {
    w.s.device = d;
    CHECK(w.call(0, 100) == KVP_OK);
  }
  Staging::Lease l[9];
  for (int k = 0; k < 8; ++k) {
    w.s.stream(k + 1);
    CHECK(w.st.lease(100, k + 1, &l[k]) == KVP_OK);
  }
  w.s.stream(9);
  CHECK(w.st.lease(100, 9, &l[8]) == KVP_EINVAL);
  for (int k = 0; k < 8; ++k) CHECK(w.st.release(l[k], true) == KVP_OK);
  CHECK(w.call(9, 100) == KVP_OK);
  w.drain();
}

}  // namespace

int main(int argc, char** argv) {
  const unsigned seed = argc > 1 ? (unsigned)std::atoi(argv[1]) : 1;
  recycled_handle();
  waits_when_behind();
  events_per_block();
  capture_refused();
  failed_launches();
  failed_launch_in_a_shared_block();
  concurrent_calls();
  for (unsigned k = 0; k < 40; ++k) random_calls(seed * 1000 + k, 300);
  std::printf("ok: staging blocks\n");
  return 0;
}
