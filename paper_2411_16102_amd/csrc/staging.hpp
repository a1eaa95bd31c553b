// Pinned host memory through which the descriptors of the calls on a context reach the device.  Plain C++ with the
// runtime as a parameter, so that the bookkeeping can be run without a device.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

namespace bs {

// words of whole 16-byte units that hold n
constexpr long whole_units(long n) { return (n + 3) / 4 * 4; }

// Rt: `Stream` and `Event` types, and functions that return 0 or an error of the runtime: create / destroy (of an
// event), alloc / release (of pinned words), record, wait (for an event), wait_all (for the device),
// capturing (whether a stream is being captured into a graph).
//
// Descriptors stand one behind the other in a half of the buffer; when one does not fit any more an event is recorded
// behind the copies out of this half (calls of a context follow one another), and the other half is taken once its own
// event has passed.  An event for every call would cost the stream 5.5 us each.
//
// A captured call reads its descriptor again with every replay of the graph, and an event that it records belongs to the
// graph.  Captured descriptors therefore stand apart, one behind the other in a ring of their own with room for five of
// the longest: the last four are there whatever the calls behind them were, and of short ones as many as the ring holds.
// Rings that became too small are kept to the end (each is at most half the size of the next).
template <class Rt>
class Staging {
  Rt rt_;
  int32_t *buf_ = nullptr;
  long half_ = 0, at_ = 0;  // words of a half; place of the next descriptor in the one being filled
  int cur_ = 0;
  typename Rt::Event ev_[2] = {};
  bool live_[2] = {};
  int32_t *kept_ = nullptr;
  long ring_ = 0, kept_at_ = 0;  // words of the ring of captured descriptors; place of the next one
  std::vector<int32_t *> outgrown_;

  int keep(long words, int32_t **out) {
    if (5 * words > ring_) {
      const long want = whole_units(std::max(2 * ring_, 5 * words));
      outgrown_.reserve(outgrown_.size() + 1);
      int32_t *bigger = nullptr;
      if (const int e = rt_.alloc(&bigger, want)) return e;
      if (kept_) outgrown_.push_back(kept_);
      kept_ = bigger;
      ring_ = want;
      kept_at_ = 0;
    } else if (kept_at_ + words > ring_) {
      kept_at_ = 0;
    }
    *out = kept_ + kept_at_;
    kept_at_ += words;
    return 0;
  }

 public:
  explicit Staging(Rt rt = Rt()) : rt_(rt) {}

  // a buffer with room for `words` in either half, a ring of `ring` words for captured descriptors
  int open(long words, long ring) {
    for (typename Rt::Event &ev : ev_)
      if (const int e = rt_.create(&ev)) return e;
    words = whole_units(words);
    ring = whole_units(ring);
    if (const int e = rt_.alloc(&buf_, 2 * words)) return e;
    if (const int e = rt_.alloc(&kept_, ring)) return e;
    ring_ = ring;
    half_ = words;
    return 0;
  }

  // (nothing may still be read from either)
  void close() {
    for (int32_t *p : {buf_, kept_})
      if (p) (void)rt_.release(p);
    for (int32_t *p : outgrown_) (void)rt_.release(p);
    for (typename Rt::Event ev : ev_)
      if (ev) (void)rt_.destroy(ev);
  }

  // the longest descriptor of a captured call that place() needs no memory for, in whole units
  long captured_room() const { return ring_ / 5 / 4 * 4; }

  // Room for `words`, a multiple of four: whole 16-byte units, on a 16-byte boundary.  They may be read by what `stream`
  // is given next.  *is_captured: whether by a graph.
  int place(long words, typename Rt::Stream stream, int32_t **out, bool *is_captured = nullptr) {
    bool captured = false;
    if (const int e = rt_.capturing(stream, &captured)) return e;
    if (is_captured) *is_captured = captured;
    if (captured) return keep(words, out);
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
