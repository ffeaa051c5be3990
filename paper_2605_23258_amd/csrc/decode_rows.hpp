// What the decode kernels and their launches compute about rows without a device, so that it runs on the host by itself.
#pragma once
#include <algorithm>
#include <cstdint>

namespace vec {

// Paged retained segments: which entry of its (sequence, head)'s block table a lane keeps for the rows row_begin ..
// row_end - 1 of a workgroup (row_begin < row_end): entry (row_begin >> block_shift) + lane, the last one of the range in the
// lanes beyond.  cap: rows the table has blocks for, at least 1.  A step's own token is row cap where the block
// is full; it has no entry (its row comes from the caller's buffers), so the range ends with the capacity for this.
constexpr int block_entry(int row_begin, int row_end, int cap, int block_shift, int lane) {
  const int last = ((row_end < cap ? row_end : cap) - 1) >> block_shift, mine = (row_begin >> block_shift) + lane;
  return mine < last ? mine : last;
}

constexpr int kMaxSplits = 64;    // of both segments together: what pick_splits keeps to, and the merge has room for

// Splits of either segment, by an estimate of the step in us.  A workgroup costs kStart, and a unit for every step_rows rows
// it reads (a retained row counts twice, an approximated one apx_cost times): kAlone by itself, kUnit when kFull workgroups or
// more share the memory.  kAtOnce run at the same time; with more, the last ones leave the chip idle for a quarter of the
// longest one.  Every split costs the merge kMerge.  The splits are divided between the segments by their cost.  Against one
// rule for all (1024 workgroups, 256 rows each at least), us: 16 sequences of 32768 tokens 70.9 -> 70.0 (768 workgroups),
// 17 of 17000 31.3 -> 26.4 (510), 3 of 2000 with eight query heads 15.3 -> 13.5; fp32, 3 of 4000 36.5 -> 20.8.
inline void pick_splits(int step_rows, int batch, int n_kv_heads, int cap_retain, int n_approx, double apx_cost, int& s_ret, int& s_apx) {
  constexpr double kStart = 4.5, kUnit = 2.3, kAlone = 0.65, kMerge = 0.08;
  constexpr int kAtOnce = 512, kFull = 300;
  const double pairs = (double)batch * n_kv_heads;
  const int steps_r = (int)(((int64_t)cap_retain + step_rows - 1) / step_rows), steps_a = (int)(((int64_t)n_approx + step_rows - 1) / step_rows);
  const double cost_r = 2.0 * steps_r, cost_a = apx_cost * steps_a;
  s_ret = steps_r > 0 || steps_a == 0 ? 1 : 0;   // nothing cached: one workgroup writes the empty partial
  s_apx = steps_a > 0 ? 1 : 0;
  if (cost_r + cost_a == 0.0) return;
  double best = -1.0;
  const int most = (int)std::min<int64_t>(kMaxSplits, (int64_t)steps_r + steps_a);
  for (int total = s_ret + s_apx; total <= most; ++total) {
    int r = (int)(total * cost_r / (cost_r + cost_a) + 0.5);
    r = std::max(steps_r > 0 ? 1 : 0, std::min({r, steps_r, total - (steps_a > 0 ? 1 : 0)}));      // r + a <= total
    const int a = std::max(steps_a > 0 ? 1 : 0, std::min(total - r, steps_a));
    const double count = pairs * (r + a), full = std::min(1.0, count / kFull), unit = kAlone + (kUnit - kAlone) * full;
    const double longest_r = r ? 2.0 * ((steps_r + r - 1) / r) : 0.0, longest_a = a ? apx_cost * ((steps_a + a - 1) / a) : 0.0;
    const double longest = kStart + unit * std::max(longest_r, longest_a);
    double t = longest;
    if (count > kAtOnce) t = std::max(t, (kStart * count + unit * pairs * (cost_r + cost_a)) / kAtOnce + 0.25 * longest);
    t += kMerge * (r + a);
    if (best < 0.0 || t < best) { best = t; s_ret = r; s_apx = a; }
    if (count > 4 * kAtOnce) break;              // more would only add starts
  }
}

}  // namespace vec
