// Pinned host memory for the work lists of calls (host code; the runtime calls it makes are Rt's, so a CPU
// test can drive it with stand-ins for streams and events).
//
// A call leases a piece, the GPU reads it (copied into device memory by `upload`, or, for metadata each wave
// reads once, read by the kernels directly over the bus: `lease` ... `release`), and the piece is written again
// only after that work.
//
// Pieces are cut from blocks; a block is closed by recording one event behind its work, and is used again once
// the event has completed.
//  * The null stream's calls share an open block per device, closed when it has no room for the next piece: an
//    event behind every call costs the stream a 5.6 us gap before its next kernel (kernel trace; no gap between
//    kernels without one): mixed decode 371.8 -> 369.1 us, RLHF 180.2 -> 177.2 us, a 67 MB append 20.7 -> 17.2 us
//    without.
//  * A call on any other stream takes a block of its own, closed when the call ends.  Such a stream can be
//    destroyed with work pending and its handle given to a new one, and an event recorded later on that handle
//    would not be behind the old stream's work; during a call the handle is the caller's.  (hipStreamPerThread,
//    another stream in every thread, is among these.)
// A capturing stream is refused: a graph would read the piece on every launch, long after it has been rewritten.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <mutex>

#include "kvpattn.h"

namespace kvp {

// Rt: types Stream (the null stream is Stream{}), Event (Event{} is none), Error (0 is success), and
//   get_device(int*), is_capturing(Stream, bool*), event_create(Event*), event_destroy(Event),
//   event_record(Event, Stream), event_done(Event) -> bool, event_wait(Event), host_alloc(void**, size_t),
//   host_free(void*), and the error sinks fail(code, format, ...) -> code and hip_fail(Error, what) -> code.
template <class Rt>
class StagingOf {
 public:
  using Stream = typename Rt::Stream;

  struct Lease {
    void* host = nullptr;
    int slot = -1;
  };

  int lease(size_t n, Stream s, Lease* out) {
    int dev = 0;
    auto e = Rt::get_device(&dev);
    if (e) return Rt::hip_fail(e, "hipGetDevice");
    const bool shared = s == Stream{};  // the null stream: never destroyed, never capturing
    if (!shared) {
      bool capturing = false;
      e = Rt::is_capturing(s, &capturing);
      if (e) return Rt::hip_fail(e, "hipStreamIsCapturing");
      if (capturing)
        return Rt::fail(KVP_EHIP, "the stream is capturing a graph, which the call's metadata would not outlive "
                        "(paged_decode_attn_noalloc can be captured)");
    }
    n = (n + 255) & ~size_t(255);
    std::lock_guard<std::mutex> lock(mu_);
    int idx = -1;
    for (int k = 0; k < kBlocks && shared && idx < 0; ++k) {
      Block& b = blocks_[k];
      if (b.state != kOpen || b.closing || b.device != dev) continue;
      if (b.used + n <= b.cap) {
        idx = k;
      } else {
        const int rc = close(&b);
        if (rc) return rc;
      }
    }
    if (idx < 0) {
      const int rc = acquire(n, dev, &idx);
      if (rc) return rc;
      Block& b = blocks_[idx];
      b.state = kOpen;
      b.stream = s;
      b.used = 0;
      b.leases = 0;
      b.closing = !shared;
    }
    Block& b = blocks_[idx];
    out->host = b.host + b.used;
    out->slot = idx;
    b.used += n;
    b.leases++;
    return KVP_OK;
  }

  // Marks the end of the call that leased the piece: the GPU work that reads it is enqueued on the stream given
  // to `lease`; after a failed launch (launched = false) perhaps only part of it, or none.
  int release(const Lease& l, bool launched) {
    std::lock_guard<std::mutex> lock(mu_);
    Block& b = blocks_[l.slot];
    b.leases--;
    if (b.leases > 0) return KVP_OK;
    int open = 0;
    for (const Block& x : blocks_) open += x.state == kOpen && !x.closing;
    if (!b.closing && open <= kMaxOpen) return KVP_OK;
    const int rc = close(&b);
    if (rc == KVP_OK || launched || b.stream == Stream{}) return rc;
    b.state = kFree;  // a call's own block: a stream that takes neither the launch nor an event has no work
    return KVP_OK;    // (the caller reports the launch)
  }

 private:
  // The start's eight concurrent calls beside the open blocks.
  static constexpr int kMaxOpen = 4;
  static constexpr int kBlocks = 8 + kMaxOpen;
  static constexpr size_t kBlockBytes = 1 << 20;
  enum State { kFree, kOpen, kPending };
  struct Block {
    unsigned char* host = nullptr;
    size_t cap = 0, used = 0;
    State state = kFree;
    Stream stream{};
    int device = -1;        // device of the event
    int leases = 0;         // calls between lease and release
    bool closing = false;   // takes no more pieces: the last release records the event
    typename Rt::Event ev{};
    uint64_t closed = 0;    // order of closing
  };

  // Record the event behind the block's work (by the last release if calls still hold pieces).  A block whose
  // event cannot be recorded is not used again: nothing tells when its pieces have been read.
  int close(Block* b) {
    b->closing = true;
    if (b->leases > 0) return KVP_OK;
    const auto e = Rt::event_record(b->ev, b->stream);
    if (e) return Rt::hip_fail(e, "hipEventRecord");
    b->state = kPending;
    b->closed = ++order_;
    return KVP_OK;
  }

  // A block of at least n bytes that nothing reads, with an event of device `dev`.
  int acquire(size_t n, int dev, int* out) {
    int best = find(n, dev);
    if (best < 0 || blocks_[best].cap < n) {  // none that fits as it is: blocks whose work has completed
      for (Block& b : blocks_)
        if (b.state == kPending && Rt::event_done(b.ev)) b.state = kFree;
      best = find(n, dev);
    }
    if (best < 0) {  // wait for the one closed first
      for (int k = 0; k < kBlocks; ++k)
        if (blocks_[k].state == kPending && (best < 0 || blocks_[k].closed < blocks_[best].closed)) best = k;
      if (best < 0) return Rt::fail(KVP_EINVAL, "more than %d concurrent calls hold metadata blocks", kBlocks);
      const auto e = Rt::event_wait(blocks_[best].ev);
      if (e) return Rt::hip_fail(e, "hipEventSynchronize(staging)");
      blocks_[best].state = kFree;
    }
    Block& b = blocks_[best];
    if (b.ev != typename Rt::Event{} && b.device != dev) {
      Rt::event_destroy(b.ev);
      b.ev = {};
    }
    if (b.ev == typename Rt::Event{}) {
      const auto e = Rt::event_create(&b.ev);
      if (e) return Rt::hip_fail(e, "hipEventCreate");
      b.device = dev;
    }
    if (n > b.cap) {
      if (b.host) Rt::host_free(b.host);
      b.host = nullptr;
      b.cap = 0;
      const size_t cap = std::max(n, kBlockBytes);
      void* p = nullptr;
      const auto e = Rt::host_alloc(&p, cap);
      if (e) return Rt::fail(KVP_ENOMEM, "hipHostMalloc(%zu): %s", cap, Rt::error_string(e));
      b.host = static_cast<unsigned char*>(p);
      b.cap = cap;
    }
    *out = best;
    return KVP_OK;
  }

  // The free block to take: one that fits on the same device, then one to allocate, then one to replace; -1 if none.
  int find(size_t n, int dev) const {
    int best = -1;
    for (int k = 0; k < kBlocks; ++k)
      if (blocks_[k].state == kFree && (best < 0 || rank(blocks_[k], n, dev) < rank(blocks_[best], n, dev))) best = k;
    return best;
  }

  static int rank(const Block& b, size_t n, int dev) {
    if (b.cap >= n) return b.device == dev ? 0 : 1;
    return b.cap == 0 ? 2 : 3;
  }

  std::mutex mu_;
  Block blocks_[kBlocks];
  uint64_t order_ = 0;
};

}  // namespace kvp
