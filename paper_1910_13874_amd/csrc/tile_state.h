// What the count arrays of a split tile's workspace hold between calls, and
// what has to be zeroed before the next one.  Host logic only.
//
// Pushes add to zeroed counts, and every tile clears what it wrote, so between
// calls the arrays are zero -- unless the array or its layout is new, a call
// failed on the way, or its tiles gathered level 2 with 16-bit copies: those
// leave level 2 as their steps wrote it, which the next such tile overwrites
// whole.  All of it follows from the calls, not from the code that enqueues
// their work, since a replayed capture runs none of that.
#pragma once
#include <cstddef>

namespace ged {

class TileState {
 public:
  struct Fill {
    bool counts = false;  // levels 1 and 2 and the worklist length
    bool level2 = false;  // level 2 alone
    bool copy = false;    // the 16-bit copy of level 1
  };

  // Levels 1, 2 and the worklist length are zero.
  bool zero() const { return zero_; }

  void counts_replaced() { zero_ = false; }
  void copy_replaced() { copy_zero_ = false; }

  // What to zero before tiles of a layout of `bytes` per level run; gathered16:
  // they gather level 2 with 16-bit copies.
  Fill fit(size_t bytes, bool gathered16) {
    Fill f;
    f.counts = !zero_ || bytes != bytes_;
    f.level2 = !f.counts && level2_left_ && !gathered16;
    f.copy = gathered16 && !copy_zero_;
    if (f.counts || f.level2) level2_left_ = false;
    if (gathered16) copy_zero_ = true;
    zero_ = true;
    bytes_ = bytes;
    return f;
  }

  // Before a call's work is launched (by capture, replay or eagerly), and once
  // it has finished; a call that fails in between never gets to end().
  void begin(bool gathered16) {
    zero_ = false;
    if (gathered16) {
      copy_zero_ = false;
      level2_left_ = true;
    }
  }
  void end(bool gathered16) {
    zero_ = true;
    if (gathered16) copy_zero_ = true;
  }

 private:
  bool zero_ = false, copy_zero_ = false, level2_left_ = false;
  size_t bytes_ = 0;
};

}  // namespace ged
