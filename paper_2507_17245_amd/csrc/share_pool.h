// Scratch buffers of one device, lent to one call at a time and kept between calls. No HIP in here: `Rt` brings
//   Stream, Event     handles
//   allocate(&ptr), deallocate(ptr), create(&event), destroy(event)
//   record(event, stream)   the event completes when all work now queued on the stream has
//   wait(stream, event)     work queued on the stream from now on starts after the event
//   done(event)             whether it has completed
//   lasting(stream)         whether the handle names one stream for as long as the process lives
// each of the others returning whether it succeeded. The caller holds a lock from lend() to give_back().
//
// A buffer is found by the stream that used it last. The handle alone proves nothing: the runtime may give the handle
// of a destroyed stream, whose work may still run, to a new one. So give_back() leaves an event behind the call's
// work, and the next call on the handle waits for it on the device (on the same live stream the order is there
// already). A stream without a buffer takes one whose event has completed, whoever used it, else a new one, so that
// the pool grows with the streams at work at the same time and not with the streams a process has ever used. A lasting
// stream keeps the buffer it got and needs no events (1 us of a decoding call's 15).
#pragma once
#include <cstddef>

namespace da {

template <typename Rt>
class SharePool {
 public:
  typedef typename Rt::Stream Stream;
  typedef typename Rt::Event Event;
  static constexpr int kMost = 16;

  // A buffer for work on `stream`, null if there is none to have. Each one lent has to be given back.
  void* lend(Stream stream) {
    for (int i = lost_; i < count_; ++i)
      if (buffers_[i].stream == stream) return Rt::lasting(stream) || Rt::wait(stream, buffers_[i].used) ? lent(i) : nullptr;
    for (int i = lost_; i < count_; ++i)
      if (!Rt::lasting(buffers_[i].stream) && Rt::done(buffers_[i].used)) {
        buffers_[i].stream = stream;
        return lent(i);
      }
    if (count_ == kMost) return nullptr;
    Buffer b = {stream, nullptr, Event()};
    if (!Rt::create(&b.used)) return nullptr;
    if (!Rt::allocate(&b.ptr)) {
      (void)Rt::destroy(b.used);
      return nullptr;
    }
    buffers_[count_++] = b;
    return b.ptr;
  }

  // The work of the call that was lent a buffer last has been queued on its stream.
  void give_back() {
    const Buffer b = buffers_[count_ - 1];
    if (Rt::lasting(b.stream) || Rt::record(b.used, b.stream)) return;
    // nothing tells when the call's work ends: the buffer is not lent again
    for (int i = count_ - 1; i > lost_; --i) buffers_[i] = buffers_[i - 1];
    buffers_[lost_++] = b;
  }

  // Frees all of them; the device is idle.
  bool clear() {
    bool ok = true;
    for (int i = 0; i < count_; ++i) {
      ok = Rt::destroy(buffers_[i].used) && ok;
      ok = Rt::deallocate(buffers_[i].ptr) && ok;
    }
    count_ = lost_ = 0;
    return ok;
  }

  bool empty() const { return count_ == 0; }

 private:
  struct Buffer {
    Stream stream;
    void* ptr;
    Event used;
  };
  Buffer buffers_[kMost];   // lost ones, then by last use, the latest at the end
  int lost_ = 0, count_ = 0;

  void* lent(int i) {
    const Buffer b = buffers_[i];
    for (; i + 1 < count_; ++i) buffers_[i] = buffers_[i + 1];
    buffers_[count_ - 1] = b;
    return b.ptr;
  }
};

}  // namespace da
