// Pinned host memory through which the descriptors of the calls on a context reach the device.  Plain C++ with the
// runtime as a parameter, so that the bookkeeping can be run without a device.
#pragma once
#include <cstdint>

namespace bs {

// words of whole 16-byte units that hold n
constexpr long whole_units(long n) { return (n + 3) / 4 * 4; }

// Rt: `Stream` and `Event` types, and functions that return 0 or an error of the runtime: create / destroy (of an
// event), alloc / release (of pinned words), record, wait (for an event), wait_all (for the device).
//
// Descriptors stand one behind the other in a half of the buffer; when one does not fit any more an event is recorded
// behind the copies out of this half (calls of a context follow one another), and the other half is taken once its own
// event has passed.  An event for every call would cost the stream 5.5 us each.
template <class Rt>
class Staging {
  Rt rt_;
  int32_t *buf_ = nullptr;
  long half_ = 0, at_ = 0;  // words of a half; place of the next descriptor in the one being filled
  int cur_ = 0;
  typename Rt::Event ev_[2] = {};
  bool live_[2] = {};

 public:
  explicit Staging(Rt rt = Rt()) : rt_(rt) {}

  // a buffer with room for `words` in either half
  int open(long words) {
    for (typename Rt::Event &ev : ev_)
      if (const int e = rt_.create(&ev)) return e;
    words = whole_units(words);
    if (const int e = rt_.alloc(&buf_, 2 * words)) return e;
    half_ = words;
    return 0;
  }

  // (nothing may still be read from it)
  void close() {
    if (buf_) (void)rt_.release(buf_);
    for (typename Rt::Event ev : ev_)
      if (ev) (void)rt_.destroy(ev);
  }

  // Room for `words`, a multiple of four: whole 16-byte units, on a 16-byte boundary.  They may be read by what `stream`
  // is given next.
  int place(long words, typename Rt::Stream stream, int32_t **out) {
    if (words > half_) {
      const long want = whole_units(words + words / 4 + 1024);  // (the second half starts on a unit too)
      int32_t *bigger = nullptr;
      if (const int e = rt_.alloc(&bigger, 2 * want)) return e;
      if (const int e = rt_.wait_all()) {
        (void)rt_.release(bigger);
        return e;
      }
      if (buf_) (void)rt_.release(buf_);
      buf_ = bigger;
      half_ = want;
      at_ = 0;
      cur_ = 0;
      live_[0] = live_[1] = false;
    } else if (at_ + words > half_) {
      if (const int e = rt_.record(ev_[cur_], stream)) return e;
      live_[cur_] = true;
      const int other = cur_ ^ 1;
      if (live_[other])
        if (const int e = rt_.wait(ev_[other])) return e;
      live_[other] = false;
      cur_ = other;
      at_ = 0;
    }
    *out = buf_ + cur_ * half_ + at_;
    at_ += words;
    return 0;
  }
};

}  // namespace bs
