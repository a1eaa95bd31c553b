// How far a call cuts the contexts of its prefill rows, given the buffers that its context holds.  Plain C++, so that the
// decisions can be run without a device.
#pragma once
#include <algorithm>
#include <limits>

namespace bs {

// Partial states of cut contexts (in rows) and words of the descriptor that a plan may have
struct CutRoom {
  long slots = std::numeric_limits<long>::max(), words = std::numeric_limits<long>::max();
};

// Cutting is optional, so it asks for nothing that the call would not get without it.  Ops, on one batch:
//   build(room)     plans, cutting into no more than `room`; 0 or an error
//   slots(), words()   of that plan: its states of cut contexts, its descriptor
//   held_slots(), held_words()        what the context's buffers hold
//   captured_words()                  the longest descriptor that a captured call places without an allocation
//   capturing()     whether the call is being captured into a graph: then nothing may be allocated
//   grow(slots, words)   makes room for so many; false where the device has none
// - Under capture contexts are cut only into what the context holds.
// - A cut that the device has no room for is not made.
template <class Ops>
int plan_within(Ops &&ops) {
  if (const int rc = ops.build(CutRoom{})) return rc;
  if (ops.slots() == 0) return 0;
  const bool held = ops.slots() <= ops.held_slots() && ops.words() <= ops.held_words();
  if (held && ops.words() <= ops.captured_words()) return 0;
  if (ops.capturing()) return ops.build(CutRoom{ops.held_slots(), std::min(ops.held_words(), ops.captured_words())});
  if (held || ops.grow(ops.slots(), ops.words())) return 0;
  return ops.build(CutRoom{0, std::numeric_limits<long>::max()});
}

}  // namespace bs
