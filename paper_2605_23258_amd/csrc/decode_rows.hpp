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

// What the estimate of a decode step is made of, in us.  A workgroup costs `start`, and for every step of its rows (step_rows of
// them) between `alone`, when little else runs, and `full`, when full_at workgroups or more share the memory and the CUs.
// at_once workgroups run at the same time; with more, the last ones leave the chip idle for `last` of the longest one.
// The merge costs `slot` for every split that a trip of its loads has room for, and `trip` for every trip.
struct SplitCosts {
  int step_rows, at_once;
  double start;
  double alone_ret, full_ret, alone_apx, full_apx;      // a step of retained rows (keys and values), of approximated ones (keys)
  double full_at, last, slot, trip;
  int per_trip, per_long_trip;           // splits: up to per_trip of them, and more
};

// Measured on 437 shapes (1 to 32 sequences of 600 to 32768 tokens, 1 to 8 KV heads with 1 to 8 query heads each, plain and rotated
// keys, contiguous and paged), each with its segments cut in all ways.  per_cu: workgroups that fit a CU, by the compiled
// kernel's registers and LDS.
//   bf16, d = 128: steps of 32 KB a tensor, two workgroups per CU; a retained step counts as two approximated ones.  Against one
//     rule for all (1024 workgroups, 256 rows each at least), us: 16 sequences of 32768 tokens 70.9 -> 70.4 (768 workgroups),
//     17 of 17000 31.3 -> 26.4 (510), 3 of 2000 with eight query heads 15.3 -> 13.5.
//   bf16, d = 64: half the bytes, three per CU; alone, a step is latency, which both kinds of rows have alike.  With the constants
//     of d = 128 in their place 16 sequences of 17000 tokens took 29.1 us, now 24.1; 24 unequal ones of up to 16000 28.0, now 25.8.
//     In the mean the choice is 1.02 times the best cut (with those of d = 128: 1.06).
//   fp32: half the bytes, and the vector unit's time, which grows with the query heads; one to five per CU.  The merge reads
//     G d / 256 elements a thread, 8 or 16 splits in a trip.  With bf16's constants, d = 128: 32 sequences of 4096 tokens,
//     four query heads, 76.6 us (four workgroups a CU where three fit), now 54; 10 of 1800, eight query heads, 51.6, now 28.3.
//     In the mean 1.04 times the best cut (1.17).
//   Approximated rows that are turned back, or rebuilt one by one, cost more than their bytes.  Rebuilt, d = 128, with the costs
//     of plain ones: 16 sequences of 32768 tokens 228 us (4 + 2 splits), now 170 (2 + 2; 206 under the one rule); one of 8192 24.6 and 19.9.
enum class ApproxRows { kPlain, kTurned, kRebuilt };
constexpr SplitCosts split_costs(bool bf16, int head_dim, int group, ApproxRows kind, int per_cu) {
  const bool turned = kind == ApproxRows::kTurned, rebuilt = kind == ApproxRows::kRebuilt;
  SplitCosts c = {};
  c.at_once = 256 * per_cu;
  if (bf16) {
    const bool wide = head_dim == 128;
    c.step_rows = 128;
    c.start = wide ? 4.5 : 5.2;
    c.alone_ret = wide ? 1.3 : 1.2; c.full_ret = wide ? 4.6 : 2.2;
    if (wide) {
      c.alone_apx = turned ? 0.65 * 2.2 : rebuilt ? 3.0 : 0.65;
      c.full_apx = turned ? 2.3 * 2.2 : rebuilt ? 6.0 : 2.3;
      c.full_at = rebuilt ? 512.0 : 300.0;
    } else {
      c.alone_apx = turned ? 1.8 : rebuilt ? 1.2 : 0.9;
      c.full_apx = turned ? 4.08 : rebuilt ? 3.2 : 2.4;
      c.full_at = 768.0;
    }
    c.last = 0.25;
    c.slot = 0.08;
    c.per_trip = c.per_long_trip = 1;
    return c;
  }
  const int elements = (group * head_dim + 255) / 256;
  c.step_rows = 4096 / head_dim;
  c.start = 7.4;
  c.alone_ret = 0.45 + 0.18 * group; c.full_ret = 3.45 + 0.35 * group;
  c.alone_apx = (0.78 + 0.24 * group) * (turned ? 1.35 : 1.0);
  c.full_apx = (4.5 + 0.9 * group) * (turned ? 1.25 : 1.0);
  c.full_at = 0.65 * c.at_once;
  c.last = 0.35;
  c.slot = 0.044 * elements; c.trip = 0.36 * ((elements + 3) / 4);
  c.per_trip = 8; c.per_long_trip = elements <= 2 ? 16 : 8;
  return c;
}

// Splits of either segment: the least of the estimate.  The splits are divided between the segments by their cost.
inline void pick_splits(const SplitCosts& c, int batch, int n_kv_heads, int cap_retain, int n_approx, int& s_ret, int& s_apx) {
  const double pairs = (double)batch * n_kv_heads;
  auto steps_of = [&](int rows) { return (int)(((int64_t)rows + c.step_rows - 1) / c.step_rows); };
  const int steps_r = steps_of(cap_retain), steps_a = steps_of(n_approx);
  s_ret = steps_r > 0 || steps_a == 0 ? 1 : 0;   // nothing cached: one workgroup writes the empty partial
  s_apx = steps_a > 0 ? 1 : 0;
  if (steps_r + (int64_t)steps_a == 0) return;
  double best = -1.0;
  const int most = (int)std::min<int64_t>(kMaxSplits, (int64_t)steps_r + steps_a);
  for (int total = s_ret + s_apx; total <= most; ++total) {
    const double shared = std::min(1.0, pairs * total / c.full_at);
    const double step_r = c.alone_ret + (c.full_ret - c.alone_ret) * shared, step_a = c.alone_apx + (c.full_apx - c.alone_apx) * shared;
    const double work = step_r * steps_r + step_a * steps_a;
    int r = (int)(total * step_r * steps_r / work + 0.5);
    r = std::max(steps_r > 0 ? 1 : 0, std::min({r, steps_r, total - (steps_a > 0 ? 1 : 0)}));      // r + a <= total
    const int a = std::max(steps_a > 0 ? 1 : 0, std::min(total - r, steps_a));
    const double count = pairs * (r + a);
    const double longest = c.start + std::max(r ? step_r * ((steps_r + r - 1) / r) : 0.0, a ? step_a * ((steps_a + a - 1) / a) : 0.0);
    double t = longest;
    if (count > c.at_once) t = std::max(t, (c.start * count + pairs * work) / c.at_once + c.last * longest);
    const int per_trip = r + a > c.per_trip ? c.per_long_trip : c.per_trip, trips = (r + a + per_trip - 1) / per_trip;
    t += (c.slot * per_trip + c.trip) * trips;
    if (best < 0.0 || t < best) { best = t; s_ret = r; s_apx = a; }
    if (count > 4.0 * c.at_once) break;          // more would only add starts
  }
}

}  // namespace vec
