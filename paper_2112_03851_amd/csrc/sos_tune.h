// The tuner's comparison of trial times (plain C++, for host tests too).
#pragma once

#include <math.h>

namespace sos {

// A candidate replaces the tuner's best only when it is faster by more than
// the launch-to-launch noise (1 %): the earliest of near-equal shapes wins, so
// repeated tunings of one problem agree.
constexpr double kTuneMargin = 0.99;

// The best candidate so far: its own time, which is what it is compared by later on.
// (Whole solves with every on-chip team size on 39 random geometries where that form
// wins: the team taken by this rule is 0.12 % slower than the best one on average, 3.2 %
// at worst; with the larger of teams within 3 % of each other 0.27 and 5.2 %.)
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
