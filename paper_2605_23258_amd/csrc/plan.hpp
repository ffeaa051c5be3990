// How a launch's work is cut into steps per workgroup.  Host code without HIP.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace vec {

// The smallest step of 1 .. most for which workgroups(step), which never grows with the step, is at most `target`; `most` if
// there is none.
template <typename F> int64_t smallest_step(int64_t most, int64_t target, F&& workgroups) {
  int64_t lo = 1, hi = most;
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (workgroups(mid) <= target) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// Routing in one launch: units of tokens per part, the fewest with which `count` sequences of n_heads heads each, their heads
// units[b] long, have no more workgroups than one per CU (or one per head).  A part takes as long as its units (rows to copy above
// all), whoever's they are: with as many parts for every head, the workgroups of eight prompts of 2048 to 8192 tokens, 8 heads, ended
// 14 to 26 us after the start, now 15 to 23.5 (their rows, 50 MB in and out, take 8 of it).
// One step after the other instead of by halving, 64 prompts of 16384 tokens, 8 heads, took the host 8.8 us per call.
inline int part_units(const int* units, int count, int n_heads) {
  const int most = *std::max_element(units, units + count);
  if ((int64_t)count * n_heads >= 256) return most;           // a part per head
  return (int)smallest_step(most, 256, [&](int64_t step) {
    int64_t parts = 0;
    for (int b = 0; b < count; ++b) parts += (units[b] + step - 1) / step;
    return parts * n_heads;
  });
}

}  // namespace vec
