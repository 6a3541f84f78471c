// The tuner's comparison of trial times (plain C++, for host tests too).
#pragma once

#include <math.h>

namespace sos {

// A candidate replaces the tuner's best only when it is faster by more than
// the launch-to-launch noise (1 %): the earliest of near-equal shapes wins, so
// repeated tunings of one problem agree.
constexpr double kTuneMargin = 0.99;

// The best candidate so far: its own time, which is what it is compared by later on.
// (Taking a larger on-chip team that is up to 3 % slower lost as often as it won: 64^3
// in 64, fours for threes, 668 ms a solve for 707, but at near-equal trials 16 x 9 x 24
// in 4, eights for sixes, 13.4 for 13.0, and 15 x 32 x 18 in 18, fours for threes,
// 23.2 for 23.0.)
struct TuneBest {
  double ms = INFINITY;
  int which = -1;
  bool offer(int candidate, double t) {
    if (!(t < ms * kTuneMargin)) return false;
    ms = t;
    which = candidate;
    return true;
  }
};

// Whether a best of one kind (the streaming form) replaces that of another, tried
// earlier (the on-chip form).
inline bool tune_replaces(const TuneBest& later, const TuneBest& earlier) {
  return later.ms < earlier.ms * kTuneMargin || !isfinite(earlier.ms);
}

}  // namespace sos
