// How a reduction's elements are split over workgroups (k_solve.hip).  Plain C++, so
// that the split can be checked on the host.
#pragma once

#include "hd.h"

namespace ahlp {

constexpr int RED_THREADS = 256;
// (240 partials and the arrival count a reduction take what 256 partials do)
constexpr int RED_PARTIALS = 240;

// Workgroups of a reduction of n elements.  Four elements a thread while there are few
// (ratios are divisions), but no more workgroups than 64 then, since their arrivals
// queue: 520 elements 9.5 -> 4.8 us a set against two launches of 256 workgroups.
// From 2^17 elements on a thread's own chain of loads and divisions is the longer
// part: workgroups of 2048 elements up to 128 of them, of 4096 past 2^19.  A step's set
// of eleven (four of them ratio tests), us in one launch of 64 workgroups, by this rule,
// and in two launches of 256 (without the gap between them): 262176 elements 19.5, 14.8,
// 17.4; 320848 24.6, 17.2, 18.8; 586820 38.2, 25.5, 24.1; 1.2 M 68.9, 40.5, 37.2; 2.2 M
// 123.5, 59.5, 58.8; six maxima of 1.2 M elements 15.8, 17.3, 17.7.
AHLP_HD int red_wgs(long long n) {
  long long w = (n + 4 * RED_THREADS - 1) / (4 * RED_THREADS);
  if (w > 64) w = 64;
  if (n > 64 * 2048) w = n / 2048 / 16 * 16;
  if (n > 128 * 2048) w = 128;
  if (n > 128 * 4096) w = n / 4096 / 16 * 16;
  return w < 1 ? 1 : w > RED_PARTIALS ? RED_PARTIALS : (int)w;
}

}  // namespace ahlp
