// Which launch sequences of an iteration the host enqueues between two polls. Host code without
// HIP, so that it can be compiled and tested by itself.
#pragma once

namespace gsi {

// Launch sequences of an iteration (launch_iteration): the full one; the short one; the full one
// before a short one, which stops the launches after it when the short one could not follow.
enum Sequence { SEQ_FULL, SEQ_LEAN, SEQ_FULL_LEAD, SEQUENCES };

// A batch: count iterations, the first with the sequence first, the others with rest.
struct Batch {
  int count;
  Sequence first, rest;
};

// The next batch between two polls. Short sequences follow a full one from any state and stop the
// launches after them where an iteration needs the full one (a hold): an explicit A X, the
// gradient's own pass after a void step. The launches behind a hold return at once, but each
// still costs its launch, up to every - 1 iterations of them. So a hold is followed by a batch of
// full sequences, which carry out such iterations in line, and each further hold without a whole
// batch of short ones between doubles their number: a solve at rounding level that holds in every
// iteration wastes every iterations of launches log2(iterations / every) times (400 iterations on
// a diagonal matrix, every 25: 150 of them; without, 24 in each iteration).
class LaunchPlan {
 public:
  // short_ok: the engine has a short sequence
  LaunchPlan(int every, bool short_ok) : every_(every), short_ok_(short_ok) {}

  // left: iterations that the cap leaves (at least one is launched)
  Batch next(int left) const {
    int count = every_;
    if (short_ok_ && full_left_ > 0 && full_left_ < count) count = full_left_;
    if (left < count) count = left;
    if (count < 1) count = 1;
    if (!short_ok_ || full_left_ > 0) return {count, SEQ_FULL, SEQ_FULL};
    return {count, lead_ ? SEQ_FULL_LEAD : SEQ_LEAN, SEQ_LEAN};
  }
  // a batch of next() has run; held: it ended in a hold
  void ran(const Batch& b, bool held) {
    if (held) {
      backoff_ = backoff_ > 0 && backoff_ < (1 << 20) ? 2 * backoff_ : every_;
      full_left_ = backoff_;
    } else if (b.rest == SEQ_LEAN) {
      backoff_ = 0;
    } else {
      full_left_ -= b.count;
    }
    lead_ = held || b.rest != SEQ_LEAN;
  }
  // the host has changed the state (the gradient is not current)
  void restart() { lead_ = true; }

 private:
  int every_;
  bool short_ok_;
  bool lead_ = true;
  int full_left_ = 0, backoff_ = 0;
};

}  // namespace gsi
