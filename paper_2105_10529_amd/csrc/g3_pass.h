// How the amplitude kernel of g g -> t t~ g g g (gg3.h) takes the gluon
// polarisation states of a chunk of events: plain C++, no device code.
#pragma once
#include <stdint.h>

namespace mf {
namespace g3 {

constexpr int GSTATES = 32;  // gluon polarisation states
constexpr int GSP = 4;       // of them in the smallest pass

// A pass takes `states` gluon states of every event of the chunk; a block
// (one wave of events) `per_block` of them in turn.
struct Pass {
  int states, per_block;
};

// Rounds of one state each that the passes over all states take on a chip that
// holds `resident` blocks at once, for a chunk of `blocks` blocks of events.
inline int64_t pass_rounds(Pass p, int64_t blocks, int64_t resident) {
  const int64_t launched = blocks * (p.states / p.per_block);
  return GSTATES / p.states * ((launched + resident - 1) / resident) * p.per_block;
}

// The pass with the fewest rounds among those of at most max_states states (or
// GSP).  A chunk that fills the chip by itself takes its GSP states in one
// block; a smaller one would leave most SIMDs idle, so it takes one block per
// state, and more states per pass where that fills the last round better.
// Equal rounds take the smaller pass, which needs less memory.  Times follow
// the rounds (what a block does once per event is a quarter of a state and
// hidden on a full chip); FP32, 1024 resident blocks, four states in a block /
// one state per block with 4, 8, 16 and 32 states per pass: 128 blocks 13.9 /
// 4.24, 2.59, 2.58, 2.53 ms; 250 blocks 14.8 / 5.17, 5.15, 4.99, 4.94 ms; 700
// blocks 18.0 / 15.0, 14.4 ms; 1024 blocks 19.7 / 19.8, 19.6 ms; 1300 blocks
// 35.7 / 28.7 ms; 2048 blocks 38.4 / 38.9 ms.
inline Pass pass_shape(int64_t blocks, int64_t resident, int64_t max_states) {
  Pass best{GSP, GSP};
  for (int s = GSP; s <= GSTATES; s *= 2) {
    const Pass p{s, 1};
    if (s > GSP && s > max_states) break;
    if (pass_rounds(p, blocks, resident) < pass_rounds(best, blocks, resident)) best = p;
  }
  return best;
}

// The pass whose buffer can be had: alloc(p) provides it or returns false, and
// then a smaller pass is tried, down to the smallest.
template <class Alloc> bool fitting_pass(int64_t blocks, int64_t resident, int64_t max_states, Alloc alloc, Pass& p) {
  for (;;) {
    p = pass_shape(blocks, resident, max_states);
    if (alloc(p)) return true;
    if (p.states == GSP) return false;
    max_states = p.states / 2;
  }
}

}  // namespace g3
}  // namespace mf
