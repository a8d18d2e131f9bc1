// What the host knows of a running device loop, and which pieces it launches ahead of it.  Plain host C++.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace jet {

// The loop (Algorithm 1) runs on the device.  One record per context holds the state its decisions need;
// small control kernels advance it between the phases of an iteration, and every kernel of a phase returns
// at once unless the record is in that phase, so the host may launch a phase before the loop is known
// to reach it.
enum LoopPhase : int32_t {
  kPhJet = 0,    // candidates, afterburner, selection and application of the kept moves
  kPhRb = 1,     // rebalancing rounds (Section 4.3)
  kPhRoll = 3,   // rollback to the best partition of the temperature round
  kPhDone = 4,
  kPhAny = -1,   // a launch outside the loop (inspection calls): never gated
};

// What the host follows of a running loop: one word per control kernel, stored by it in pinned memory.
struct LoopMail {
  uint32_t seq;       // low kMailSeqBits bits of LoopCtl::seq
  int32_t mask;       // phases the record (a union: any of its hypergraphs) is in
  int32_t phase;      // the lowest of them
  int32_t rb_rounds;  // of the current iteration, once the next Jet phase runs of the last one (clipped)
  bool last;          // the round ends with the current iteration unless that improves
  bool err;           // a kernel reported an error
};
constexpr int kMailSeqBits = 24, kMailMaskSh = 24, kMailMaskBits = 5;
constexpr int kMailRbSh = 29, kMailRbBits = 16, kMailLastSh = 45, kMailErrSh = 46;
constexpr uint32_t kMailSeqMask = (1u << kMailSeqBits) - 1u;
inline LoopMail read_mail(unsigned long long w) {
  const int32_t mask = (int32_t)((w >> kMailMaskSh) & ((1u << kMailMaskBits) - 1u));
  return LoopMail{(uint32_t)w & kMailSeqMask, mask, mask ? __builtin_ctz((unsigned)mask) : 0,
                  (int32_t)((w >> kMailRbSh) & ((1u << kMailRbBits) - 1u)), ((w >> kMailLastSh) & 1u) != 0,
                  ((w >> kMailErrSh) & 1u) != 0};
}

// The pieces in flight and the next one to launch: the one of the phase the loop is in, then up to `lead` in
// all of those that are likely to follow.  The number of rebalancing rounds of an iteration is guessed
// from the number of the iteration before it (what followed that number last time); the guess is acted on
// while the last one of its kind was right.
class Ahead {
 public:
  Ahead(bool rb_only_, int32_t lead_) : rb_only(rb_only_), lead(lead_) {
    std::fill(sure, sure + kKinds, true);
    m.phase = rb_only ? kPhRb : kPhJet;  // before the first report, what it is likely to say
    launched(kPhAny, 1);                 // the set-up's control kernel reports too
  }

  LoopMail m{};       // the last report
  uint32_t seen = 0;  // its number
  bool done() const { return m.phase == kPhDone || m.err; }

  // phase of the piece to launch next, -1: wait for a report
  int32_t want() const {
    int32_t i = (int32_t)(std::find(flight, flight + n, m.phase) - flight);
    if (i == n) return m.phase;
    if (n >= lead) return -1;
    LoopMail at = m;
    for (int32_t before = prev;; ) {  // along the pieces behind the current one, as far as they are as foreseen
      const int32_t ph = follows(at, before);
      if (++i == n) return ph;
      if (ph != flight[i]) return -1;
      if (ph == kPhJet) before = at.phase == kPhRb ? at.rb_rounds + 1 : 0;
      at.rb_rounds = ph == kPhRb && at.phase == kPhRb ? at.rb_rounds + 1 : 0;
      at.last = at.last && ph != kPhJet;
      at.phase = ph;
    }
  }
  // its control kernels (reports) fit the list
  bool room(int32_t reports) const { return n + reports <= kMost; }
  void launched(int32_t phase, int32_t reports) {
    for (int32_t i = 0; i < reports; ++i) flight[n++] = phase;
  }
  int32_t in_flight() const { return n; }

  void report(const LoopMail &now) {
    const int32_t was = m.phase;
    const int32_t got = std::min<int32_t>((int32_t)((now.seq - seen) & kMailSeqMask), n);
    bool ran = false;  // a piece of the phase we knew of has run
    for (int32_t i = 0; i < got; ++i) ran = ran || flight[i] == was;
    std::copy(flight + got, flight + n, flight);
    n -= got;
    m = now;
    seen = now.seq;
    if (ran && !rb_only && was != kPhRoll && m.phase != kPhRb) learn(m.rb_rounds);
  }

 private:
  static constexpr int kKinds = 17;   // rounds of the iteration before: 0..15, more
  static constexpr int kMost = 256;   // control kernels in flight at most
  int32_t guess[kKinds] = {};
  bool sure[kKinds];
  int32_t prev = 0;  // rounds of the last finished iteration
  bool rb_only;      // rebalancing alone: another round is the likely thing
  int32_t lead;
  int32_t flight[kMost], n = 0;  // phases of the launched control kernels that have not reported, oldest first

  static int slot(int32_t rounds) { return std::min<int32_t>(rounds, kKinds - 1); }
  // an iteration with this many rounds has ended
  void learn(int32_t rounds) {
    const int s = slot(prev);
    sure[s] = guess[s] == rounds;
    guess[s] = rounds;
    prev = rounds;
  }
  // the phase after the one at stands for, in an iteration after one of `before` rounds; -1: wait and see
  int32_t follows(const LoopMail &at, int32_t before) const {
    if (rb_only) return kPhRb;
    const int s = slot(before);
    if (at.phase == kPhJet) {
      if (!sure[s]) return -1;
      if (guess[s] > 0) return kPhRb;
      return at.last ? -1 : kPhJet;
    }
    if (at.phase == kPhRb) {
      if (at.rb_rounds + 1 < guess[s]) return kPhRb;
      if (at.rb_rounds + 1 == guess[s] && sure[s] && !at.last) return kPhJet;
    }
    return -1;
  }
};

}  // namespace jet
