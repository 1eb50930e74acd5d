// scratch.hpp -- a handle's device scratch: stream-ordered blocks kept between
// calls.  Internal to libmpdd.
//
// A call takes a block on its stream and gives it back on the same stream.
// Blocks come from the handle's memory pool; up to KEEP of them stay with the
// handle afterwards, since an allocation and a free on the pool cost the host
// 9 to 11 us a call, four kernel launches' worth (taking and giving back a
// kept block: 2.7 us).  An event recorded when a block is given back orders
// its next use after its last one, whatever the streams: a block last used on
// the caller's own stream is taken first (the wait is then in order), one of
// another stream only once its work is done, so that calls on different
// streams do not wait for each other.  Free blocks are given back to the pool,
// those unused for longest first, when there are more than KEEP of them or they
// hold more than KEEP_BYTES (one block may hold more by itself: a call that
// needs it would need it again); when one of the caller's stream is too small;
// when an allocation that a call cannot do without fails; and with the handle.  A
// stream under capture uses the pool itself (its allocations become graph nodes).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <mutex>
#include <new>
#include <vector>

namespace mpdd {

class ScratchCache {
 public:
  static constexpr size_t KEEP_BYTES = (size_t)8 << 30;

  void open(hipMemPool_t pool) { pool_ = pool; }

  // `bytes` bytes for work enqueued on st until put(): *p, or an error with no
  // error left pending.  `optional`: the caller can do without, so that where there
  // is no memory nothing is given up or waited for; and after a failed allocation
  // the next RETRY requests that would make one as large fail at once (a failed
  // one takes the driver as long as a call).
  hipError_t get(void** p, size_t bytes, hipStream_t st, bool optional = false) {
    if (capturing(st)) return pool_alloc(p, bytes, st);
    std::lock_guard<std::mutex> lk(mu_);
    Block* own = nullptr;             // the best fit among st's, else its largest
    Block* other = nullptr;
    for (Block& b : blocks_) {
      if (b.busy) continue;
      if (b.stream == st) {
        if (!own || (own->bytes < bytes ? b.bytes > own->bytes
                                        : b.bytes >= bytes && b.bytes < own->bytes))
          own = &b;
      } else if (b.bytes >= bytes && (!other || b.bytes < other->bytes) && idle(b)) {
        other = &b;
      }
    }
    if (own && own->bytes >= bytes) {
      // (the event, not the handle's value, is the order: a destroyed
      // stream's handle may come back)
      const hipError_t e = hipStreamWaitEvent(st, own->done, 0);
      if (e != hipSuccess) return cleared(e);
      return take(*own, p, st);
    }
    if (other) return take(*other, p, st);
    if (optional && bytes >= refused_ && wait_ > 0) {
      --wait_;
      return hipErrorOutOfMemory;
    }
    const size_t too_small = own ? (size_t)(own - blocks_.data()) : blocks_.size();
    if (own && !optional) drop(too_small, st);
    Block b;
    b.bytes = round_size(bytes);
    hipError_t e = pool_alloc(&b.ptr, b.bytes, st);
    if (optional && e != hipSuccess) {
      refused_ = bytes;
      wait_ = RETRY;
      return e;
    }
    if (own && optional) drop(too_small, st);
    if (e != hipSuccess) {
      // hand every free block back and try once more, for the bare size
      for (size_t i = blocks_.size(); i-- > 0;)
        if (!blocks_[i].busy) drop(i, st);
      (void)hipStreamSynchronize(st);
      b.bytes = bytes;
      e = pool_alloc(&b.ptr, b.bytes, st);
      if (e != hipSuccess) return e;
    }
    {
      Relaxed relaxed;
      e = hipEventCreateWithFlags(&b.done, hipEventDisableTiming);
    }
    if (e == hipSuccess) {
      try {
        blocks_.push_back(b);
      } catch (const std::bad_alloc&) {        // (none may leave a C entry point)
        (void)hipEventDestroy(b.done);
        e = hipErrorOutOfMemory;
      }
    }
    if (e != hipSuccess) {
      (void)hipFreeAsync(b.ptr, st);
      return cleared(e);
    }
    return take(blocks_.back(), p, st);
  }

  // The work on st so far is the last to use p.  (No error left pending.)
  hipError_t put(void* p, hipStream_t st) {
    if (!p) return hipSuccess;
    std::lock_guard<std::mutex> lk(mu_);
    size_t at = blocks_.size(), count = 0, bytes = 0;
    for (size_t i = 0; i < blocks_.size(); ++i) {
      if (blocks_[i].ptr == p) at = i;
      if (blocks_[i].ptr == p || !blocks_[i].busy) {
        ++count;
        bytes += blocks_[i].bytes;
      }
    }
    if (at == blocks_.size()) return cleared(hipFreeAsync(p, st));   // taken under capture
    // (in the order of their last use)
    std::rotate(blocks_.begin() + at, blocks_.begin() + at + 1, blocks_.end());
    Block& b = blocks_.back();
    hipError_t e = hipEventRecord(b.done, st);
    b.busy = false;
    auto over = [&] { return count > KEEP || (count > 1 && bytes > KEEP_BYTES); };
    if (e == hipSuccess) {
      // the oldest ones whose work is done (the others' streams are not waited for)
      for (size_t i = 0; over() && i + 1 < blocks_.size();) {
        if (blocks_[i].busy || !idle(blocks_[i])) {
          ++i;
          continue;
        }
        --count;
        bytes -= blocks_[i].bytes;
        (void)release(i, st);
      }
      if (!over()) return hipSuccess;
    }
    const hipError_t f = release(blocks_.size() - 1, st);
    return cleared(e != hipSuccess ? e : f);
  }

  // Every block back to the pool (no call in flight).
  void close() {
    std::lock_guard<std::mutex> lk(mu_);
    for (Block& b : blocks_) {
      (void)hipEventSynchronize(b.done);
      (void)hipEventDestroy(b.done);
      (void)hipFreeAsync(b.ptr, nullptr);
    }
    blocks_.clear();
  }

  static bool capturing(hipStream_t st) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) (void)hipGetLastError();
    return cap != hipStreamCaptureStatusNone;
  }

 private:
  static constexpr size_t KEEP = 8;
  static constexpr int RETRY = 64;
  struct Block {
    void* ptr = nullptr;
    size_t bytes = 0;
    hipStream_t stream = nullptr;     // of its last use
    hipEvent_t done = nullptr;        // recorded after its last use
    bool busy = false;
  };

  // Another stream of the program may be under capture in a mode that refuses
  // queries and the like: this thread's calls here are none of that graph's.
  struct Relaxed {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  };

  static bool idle(const Block& b) {
    Relaxed relaxed;
    const bool done = hipEventQuery(b.done) == hipSuccess;
    if (!done) (void)hipGetLastError();      // (hipErrorNotReady)
    return done;
  }

  // sizes in steps of an eighth of their power of two, so that calls of
  // nearby sizes share blocks
  static size_t round_size(size_t bytes) {
    size_t step = (size_t)1 << 16;
    while (step * 16 < bytes) step *= 2;
    return (bytes + step - 1) / step * step;
  }

  // An error that this class reports itself: a later launch's check must not
  // find it again.
  static hipError_t cleared(hipError_t e) {
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
  }

  hipError_t pool_alloc(void** p, size_t bytes, hipStream_t st) {
    return cleared(hipMallocFromPoolAsync(p, bytes, pool_, st));
  }

  hipError_t take(Block& b, void** p, hipStream_t st) {
    b.busy = true;
    b.stream = st;
    *p = b.ptr;
    return hipSuccess;
  }

  // Block i (free) back to the pool, after its last use.
  void drop(size_t i, hipStream_t st) {
    Block& b = blocks_[i];
    if (cleared(hipStreamWaitEvent(st, b.done, 0)) != hipSuccess)
      (void)hipEventSynchronize(b.done);
    (void)release(i, st);
  }

  // Block i back to the pool: its work is done, or enqueued on st.
  hipError_t release(size_t i, hipStream_t st) {
    const hipError_t e = hipFreeAsync(blocks_[i].ptr, st);
    (void)hipEventDestroy(blocks_[i].done);
    blocks_.erase(blocks_.begin() + i);
    return e;
  }

  std::mutex mu_;
  hipMemPool_t pool_ = nullptr;
  std::vector<Block> blocks_;
  size_t refused_ = 0;                // bytes of the last optional allocation that failed
  int wait_ = 0;                      // requests of that size left to fail at once
};

}  // namespace mpdd
