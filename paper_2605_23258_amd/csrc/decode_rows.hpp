// What the decode kernels and their launches compute about rows without a device, so that it runs on the host by itself.
#pragma once
#include <algorithm>
#include <cmath>
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
// them) between `alone`, when little else runs, and `full`, when the chip is full: by how many workgroups there are, of full_at,
// and for the share by_cu by how many a CU has, of per_cu.  256 per_cu run at the same time; with more, the last ones leave the chip
// idle for `last` of the longest one, and the more (`idle`) the emptier the last round of workgroups is.
// The merge costs `slot` for every split that a trip of its loads has room for, and `trip` for every trip.
struct SplitCosts {
  int step_rows, per_cu;
  double start;
  double alone_ret, full_ret, alone_apx, full_apx;      // a step of retained rows (keys and values), of approximated ones (keys)
  double full_at, by_cu, last, idle, slot, trip;
  int per_trip, per_long_trip;           // splits: up to per_trip of them, and more
  bool one_round;                        // pick_one_round first
};

enum class ApproxRows { kPlain, kTurned, kRebuilt };

// Measured on 937 shapes (1 to 32 sequences of 600 to 32768 tokens, 1 to 8 KV heads, every number of query heads, plain and rotated
// keys, contiguous and paged), each with its segments cut in all ways.  per_cu: workgroups that fit a CU, by the compiled
// kernel's registers and LDS.  In the mean, times the best cut: with one rule for all kernels (1024 workgroups, 256 rows each
// at least; other kernels then), with the constants of bf16 and d = 128 for all, and now:
//   bf16, d = 128   1.35  1.08  1.08   32 KB a tensor and step, two workgroups per CU.  Constants fitted to all these shapes alike
//                                      would gain 4 % in the mean and lose 2 to 12 % on the longest, so those of before stay.
//   bf16, d = 64    1.27  1.07  1.03   half the bytes, three per CU; alone, a step is latency, which both kinds of rows have alike
//   fp32            1.35  1.17  1.03   half the bytes, and the vector unit's time, which grows with the query heads; one to five per CU
// Single shapes, us: fp32, d = 128, 32 sequences of 4096 tokens, four query heads 52 / 77 (four workgroups a CU where three fit) /
// 54; 10 of 1798, eight query heads 42 / 52 / 28; bf16, d = 64, 16 of 17000 32 / 29 / 24; bf16, d = 128, 16 of 32768 70.9 / 70.4 / 70.4
// (64.4 in one round, see pick_one_round).  The fp32 kernels of 128 dims have fewer registers since, and one more of them fits a CU.
// Approximated rows that are turned back, or rebuilt one by one, cost more than their bytes.  Rebuilt, d = 128, with the costs of
// plain ones: 16 sequences of 32768 tokens 228 us (4 + 2 splits), now 169 (2 + 2; 205 under the one rule); one of 8192 24.6 and 19.2.
constexpr SplitCosts split_costs(bool bf16, int head_dim, int group, ApproxRows kind, int per_cu) {
  const bool turned = kind == ApproxRows::kTurned, rebuilt = kind == ApproxRows::kRebuilt;
  SplitCosts c = {};
  c.per_cu = per_cu;
  c.per_trip = c.per_long_trip = 1;
  if (bf16 && head_dim == 128) {
    c.step_rows = 128;
    c.start = 4.5;
    c.alone_ret = 1.3; c.full_ret = 4.6;
    c.alone_apx = turned ? 1.43 : rebuilt ? 3.0 : 0.65; c.full_apx = turned ? 5.06 : rebuilt ? 6.0 : 2.3;
    c.full_at = rebuilt ? 512.0 : 300.0;
    c.last = 0.25;
    c.slot = 0.08;
    c.one_round = true;
  } else if (bf16) {
    c.step_rows = 128;
    c.start = 5.0;
    c.alone_ret = 1.3; c.full_ret = 0.95 * per_cu;
    c.alone_apx = turned ? 2.2 : rebuilt ? 2.0 : 1.3; c.full_apx = (turned ? 2.04 : rebuilt ? 1.4 : 1.2) * per_cu;
    c.full_at = 256.0 * per_cu;
    c.last = 0.3;
    c.slot = 0.12;
  } else {
    const int elements = (group * head_dim + 255) / 256;         // of a thread of the merge, four at a time
    // Three query heads at 128 dims: four fit by their registers (121), but what four of them take is no less than what three do.  Cut for three /
    // four, eight heads: 16 sequences of 1000 + 1000 rows 46.6 / 52.5 us a step, 24 65.2 / 70.6, 8 of 800 + 200 21.9 / 27.6, 24 of 200 + 800 33.5 / 38.9;
    // 43 shapes in the mean 4 % less, at worst (14 of 200 + 800) 30.0 / 27.1.  With more heads the cuts for as many as fit are the better ones:
    // five, 24 of 400 + 400 52.6 (two) / 43.1 (three), ten, 16 of 1000 + 1000 288 (one) / 164 (two).
    if (head_dim == 128 && group == 3) c.per_cu = per_cu = std::min(per_cu, 3);
    c.step_rows = 4096 / head_dim;
    c.start = 7.5;
    c.alone_ret = 0.9 + 0.13 * group; c.full_ret = (2.75 + 0.11 * group) * per_cu;
    c.alone_apx = (1.15 + 0.2 * group) * (turned ? 1.65 : 1.0); c.full_apx = (3.5 + 0.2 * group) * (turned ? 1.45 : 1.0) * per_cu;
    c.full_at = 0.85 * 256 * per_cu; c.by_cu = 0.15;
    c.last = 0.3; c.idle = 0.1;
    c.slot = 0.03 * elements; c.trip = 0.25 * ((elements + 3) / 4);
    c.per_trip = 8; c.per_long_trip = elements <= 2 ? 16 : 8;
  }
  return c;
}

// Splits of either segment: the least of the estimate.  The splits are divided between the segments by their cost.
inline void pick_splits(const SplitCosts& c, int batch, int n_kv_heads, int cap_retain, int n_approx, int& s_ret, int& s_apx) {
  const double pairs = (double)batch * n_kv_heads, at_once = 256.0 * c.per_cu;
  auto steps_of = [&](int rows) { return (int)(((int64_t)rows + c.step_rows - 1) / c.step_rows); };
  const int steps_r = steps_of(cap_retain), steps_a = steps_of(n_approx);
  s_ret = steps_r > 0 || steps_a == 0 ? 1 : 0;   // nothing cached: one workgroup writes the empty partial
  s_apx = steps_a > 0 ? 1 : 0;
  if (steps_r + (int64_t)steps_a == 0) return;
  double best = -1.0;
  const int most = (int)std::min<int64_t>(kMaxSplits, (int64_t)steps_r + steps_a);
  for (int total = s_ret + s_apx; total <= most; ++total) {
    const double all = pairs * total;
    const double shared = (1.0 - c.by_cu) * std::min(1.0, all / c.full_at) + c.by_cu * std::min(1.0, std::ceil(all / 256.0) / c.per_cu);
    const double step_r = c.alone_ret + std::max(0.0, c.full_ret - c.alone_ret) * shared;
    const double step_a = c.alone_apx + std::max(0.0, c.full_apx - c.alone_apx) * shared;
    const double work = step_r * steps_r + step_a * steps_a;
    int r = (int)(total * step_r * steps_r / work + 0.5);
    r = std::max(steps_r > 0 ? 1 : 0, std::min({r, steps_r, total - (steps_a > 0 ? 1 : 0)}));      // r + a <= total
    const int a = std::max(steps_a > 0 ? 1 : 0, std::min(total - r, steps_a));
    const double count = pairs * (r + a), rounds = count / at_once;
    const double longest = c.start + std::max(r ? step_r * ((steps_r + r - 1) / r) : 0.0, a ? step_a * ((steps_a + a - 1) / a) : 0.0);
    double t = longest;
    if (rounds > 1.0) t = std::max(t, (c.start * count + pairs * work) / at_once + (c.last + c.idle * (std::ceil(rounds) - rounds)) * longest);
    const int per_trip = r + a > c.per_trip ? c.per_long_trip : c.per_trip, trips = (r + a + per_trip - 1) / per_trip;
    t += (c.slot * per_trip + c.trip) * trips;
    if (best < 0.0 || t < best) { best = t; s_ret = r; s_apx = a; }
    if (rounds > 4.0) break;                     // more would only add starts
  }
}

// Splits that make one round of workgroups, or one piece of either segment for many sequences; at least least_ret of them for the retained segment.  For plain rows of 128 dims in bf16,
// whose launch puts the retained pieces of all sequences first, the approximated ones behind them: the workgroups of a CU,
// half a grid apart, are then one of each where there are as many of both, and every XCD has both kinds.  (In the order (split,
// head, sequence) an XCD has one split of eight, often all retained or all approximated.)  What a round takes: its bytes, or the steps
// of its longest piece, twice as long each where CUs have two; the merge; and something for the last pieces to end.
// A step, us, the estimate of before in its order / these / these in that order:
//   16 sequences of 32768 tokens 70.6 (4 + 2) / 64.4 (2 + 2) / 71.4; 13 66.7 (2 + 1) / 56.6; 10 48.9 / 45.7 / 50.3; 4 23.0 / 22.3;
//   24 of 16000 64.4 / 55.1 / 62.8; 32 of 8000 44.7 / 39.8 / 42.8; 64 of 8000 73.8 / 73.9; 1 of 8192 11.4 / 10.3.
//   One of 16000, eight heads, cut into 6 / 11 / 21 and about as many: 14.6 / 12.6 / 13.5; two of 8192, 4 / 6 / 12: 13.2 / 11.9 / 12.7.
//   Four times as many approximated rows as retained ones 75.2 / 70.9; four times as many retained ones 93.3 / 97.7 (26.7 / 27.1 for nine
//   sequences of 12000): more than three times as many are left to the estimate.  Rotated keys (approximated rows are vector
//   work) 69.2 / 82, and rows of 64 dims 37.1 / 37.5, 30.8 / 32.9, 14.7 / 14.7: the estimate.
// With more (sequence, head) pairs than half a round it is one piece of either segment each, and the order is all there is to choose.  A few
// workgroups beyond a round end alone: up to half a round more is left to the estimate, and all where the retained segment is the longer by
// half.  The estimate / these in that order, eight heads, retained + approximated rows, 256 more of capacity:
//   2000 + 2000: 33 sequences 89.3 / 99.0, 40 96.2 / 104.3 (with 344 to 383 pairs, 43 110.1 / 107.5 is given up); 48 117.0 / 113.2, 64 146.6 / 143.2, 65 152.8 / 160.1, 96 216.2 / 209.9;
//   700 + 700: 33 41.2 / 43.4, 43 47.0 / 47.8; 52 54.3 / 50.8, 64 61.7 / 59.2, 128 112.0 / 109.0; 1200 + 2400: 36 79.8 / 84.5; 48 99.4 / 94.6, 64 115.8 / 116.5, 80 157.5 / 151.6;
//   2400 + 1200: 36 88.7 / 94.1, 48 111.0 / 113.5, 64 142.3 / 146.8, 96 211.4 / 212.7.
// Inside a round, one piece each with the approximated one longer by half: left to the estimate where that comes to one piece each as well
// (1600 + 3500: 28 75.7 / 80.3, 32 85.1 / 87.2; 1000 + 3000: 28 63.2 / 65.3, 32 67.4 / 67.7; but 24, which it cuts finer, 63.2 / 61.0), and where
// less than three quarters of a round would run (1600 + 3500: 22 67.9 / 71.4, one query head 65.2 / 70.5, 23 71.0 / 72.1; 1000 + 3000: 22 58.2 / 57.9).
inline bool pick_one_round(const SplitCosts& c, int batch, int n_kv_heads, int cap_retain, int n_approx, int least_ret, int& s_ret, int& s_apx) {
  const int64_t steps_r = ((int64_t)cap_retain + c.step_rows - 1) / c.step_rows, steps_a = ((int64_t)n_approx + c.step_rows - 1) / c.step_rows;
  if (steps_r == 0 || steps_a == 0 || steps_r > 3 * steps_a) return false;
  const int64_t pairs = (int64_t)batch * n_kv_heads, at_once = 256 * c.per_cu;
  if (2 * pairs > at_once && (4 * pairs < 3 * at_once || 2 * steps_r > 3 * steps_a)) return false;
  const int most = (int)std::max<int64_t>(2, std::min<int64_t>(kMaxSplits, at_once / pairs));
  const double bytes = (double)pairs * (0.0121 * (double)steps_r + 0.0061 * (double)steps_a);      // us at 5.4 TB/s
  double best = -1.0;
  for (int r = std::max(1, least_ret); r < most && r <= steps_r; ++r) {
    const int64_t long_r = (steps_r + r - 1) / r;
    // as many as bring the approximated segment's pieces down to the retained one's, if there are that many
    int64_t a = std::min<int64_t>(std::min<int64_t>(most - r, steps_a), (steps_a + long_r - 1) / long_r);
    const int64_t long_a = (steps_a + a - 1) / a;
    a = (steps_a + long_a - 1) / long_a;
    const double longest = (double)std::max(long_r, long_a);
    const double t = std::max(bytes, (pairs * (r + a) > 256 ? 2.8 : 1.4) * longest) + 0.15 * longest + 0.05 * (double)(r + a);
    if (best < 0.0 || t < best) { best = t; s_ret = r; s_apx = (int)a; }
  }
  if (best >= 0.0 && 2 * pairs <= at_once && s_ret + s_apx == 2 && 2 * steps_a > 3 * steps_r) {
    int r = 1, a = 1;
    if (8 * pairs >= 3 * at_once) pick_splits(c, batch, n_kv_heads, cap_retain, n_approx, r, a);
    if (r + a == 2) return false;
  }
  return best >= 0.0;
}

// Sequences of different lengths, whose live rows only the device knows, cut by a plan that the split launch makes (PlannedSplits in
// decode_attn.hip): granules of 32 rows, four to a step; what the change to another segment costs, in granules (fitted to the workgroups'
// ends: 0.5 us a granule with the chip full, 5 a change; 4, 6 and 9 measured); and how long a line of granules may be.
constexpr int kLogGranule = 5, kStepGranules = 4, kPieceGranules = 6, kMaxPlanned = 64, kMaxPlanUnits = 1 << 28;
constexpr float kPlanTurned = 1.86f;   // a granule of approximated rows that are turned back, in plain ones
// As many workgroups as run at the same time.  Their partials, and one more for every segment, of which there are two per (sequence,
// head), are to fit kMaxSplits per pair.
constexpr int plan_workgroups(int per_cu, int pairs) { return 256 * per_cu < (kMaxSplits - 2) * pairs ? 256 * per_cu : (kMaxSplits - 2) * pairs; }
// What the workgroups of a plan compute; `inverse` is that of the float named, one step off at most.
// A line of rows is a sequence of segments, each as long as its granules and kPieceGranules for the change to it.
constexpr int plan_granules(int rows, int log_rows) { return (int)(((unsigned)rows + (1u << log_rows) - 1u) >> log_rows); }
constexpr int plan_length(int granules) { return granules > 0 ? kPieceGranules + granules : 0; }
// whether a line could be too long, `longest` the length of its longest segment: then granules are twice as long
constexpr bool plan_too_long(float longest, int batch, int n_kv_heads, int log_rows) {
  return longest * (float)batch * (float)n_kv_heads >= (float)kMaxPlanUnits && log_rows < 30;
}
// The most workgroups for the retained line where there are approximated rows: all but one of every CU's, so that each CU has at most
// so many pieces of two tensors (workgroups that are a CU's lie 256 apart).  Shares by work alone are slower however uneven the lines, also with one
// piece of approximated rows in all, and so for them the retained line's are the longest.  A step of unequal sequences, us:
//   128 dims, two per CU, 24 of 3200 rows, retained : approximated 1.3, 2, 3.5, 6 and 32 approximated rows in all: at most half 39.4, 41.9, 43.6, 44.6, 46.1; at most three
//     quarters 43.9, 45.0, 46.2, 48.2, 50.0; by work alone 43.9, 45.0, 46.2, 47.2, 52.7; as many splits for every sequence 44.3, 47.8, 45.6, 46.9, 49.9.  (At 1 and below
//     the work gives less than half.)  Rotated 44.4, 45.7, 44.5, 46.3, 46.5; 44.3, 45.7, 48.9, 49.5, 50.4; 44.4, 45.7, 49.0, 49.4, 50.6; 50.2, 49.5, 49.7, 47.7, 49.1.
//   64 dims, three per CU, 40 of 3200 rows at 2, 3.5, 6, 30: half 37.3, 37.8, 39.5, 41.4; two thirds 35.9, 36.3, 38.2, 39.7; three quarters 35.9, 38.8, 41.2, 44.2; as many splits
//     34.1, 36.8, 38.7, 40.2.  64 of 1700: 31.7, 34.8, 35.6, 37.9; 31.1, 32.3, 33.2, 35.2; 31.1, 34.4, 35.5, 38.5; 29.7, 31.9, 33.1, 35.8.  A few more than half are no
//     gain (24 of 1600 at 1 and the step's token 23.5 / 23.9; at 1.3 25.2 / 25.5, at 1.5 35.1 / 35.2): from three fifths of the work on.
constexpr int plan_most_retained(int per_cu, int wgs) { return per_cu > 2 ? wgs / per_cu * (per_cu - 1) : wgs / 2; }
// Workgroups of the retained line: by the lines' work.  inverse: of total_r + total_a * apx
constexpr int plan_retained(int wgs, int most, int total_r, int total_a, float inverse) {
  const int by_work = (int)((float)wgs * (float)total_r * inverse + 0.5f), limit = 5 * by_work > 3 * wgs ? most : wgs / 2;
  const int wgs_r = total_a > 0 ? (by_work < limit ? by_work : limit) : wgs;
  return total_r > 0 && wgs_r < 1 ? 1 : wgs_r;
}
// A workgroup's share of its line: an even one, rounded up, and by as much as its float may be below it; no more than half of kMaxSplits for
// a segment.  inverse: of the line's workgroups
constexpr int plan_share(int total, float longest, float inverse) {
  const float even = (float)total * 1.000001f * inverse, least = longest * (1.f / (float)(kMaxSplits / 2 - 2));
  const int share = (int)(even > least ? even : least) + 1;
  return share > kStepGranules ? share : kStepGranules;
}
// The head whose segment a place lies in, `offset` from where its sequence begins.  inverse: of the segment's length
constexpr int plan_head(int offset, int length, float inverse) {
  const int h = (int)((float)offset * inverse), not_after = h * length > offset ? h - 1 : h;           // at most one off
  return (not_after + 1) * length <= offset ? not_after + 1 : not_after;
}
// Granules first .. last - 1 of a segment of n that begins at `at` fall to the workgroup whose share begins at lo
struct PlanPiece { int first, last; };
constexpr PlanPiece plan_piece(int at, int n, int lo, int share) {
  const int zero = at + kPieceGranules;         // where granule 0 begins
  return {lo > zero ? lo - zero : 0, lo + share - zero < n ? lo + share - zero : n};
}
// Where the partial of workgroup `id` goes, `pair` the (sequence, head): a share has room for a step of granules, so a segment's
// workgroups are next to each other; of how many partials a segment has the workgroup with granule 0 knows
constexpr int plan_place(int id, int pair, bool is_apx, int pairs) { return id + pair + (is_apx ? pairs : 0); }
constexpr int plan_partials(int at, int n, int lo, int share) { return (at + kPieceGranules + n - 1) / share - lo / share + 1; }
// Rows of a sequence's segment.  Where the call itself says that it has none, the segment may have no memory (nor W, with no
// approximated rows), and is left out whatever the sequence's own count says, as where every sequence gets as many splits.
constexpr int planned_rows(int of_call, int of_sequence) { return of_call > 0 && of_sequence > 0 ? of_sequence : 0; }
// A lane per sequence; and enough steps of rows for the launch's workgroups (every sequence counted as the longest), since a plan costs
// a workgroup about a step, and small launches end when their one or two steps do, however they are cut.  Measured on one in which the longest
// sequence has four times the shortest one's rows, retained : approximated rows 1/6 to 6, as many splits for every sequence / a plan, us:
//   128 dims, from three steps per workgroup: 6 sequences of 4000 rows 20.5 / 19.9 (rotated 26.1 / 23.5), 16 of 3200 28.1 / 26.9 (36.6 / 32.3), 12 of 8000 48.0 / 45.0
//     (59.2 / 49.9); in the mean of 60 shapes of three to four steps 4 % less, at worst 5 % more (16 query heads: 9 %).  Below: 2 of 1700 11.1 / 13.1 (13.1 / 14.9), two heads,
//     4 of 8000 13.9 / 16.5 (18.1 / 20.5), 6 of 1700 9.9 / 12.5; 3 of 3200 13.8 / 15.3 (but rotated 19.0 / 17.2).
//   64 dims, plain, from six: 10 of 8000 26.5 / 25.5, 12 30.1 / 27.7, 28 of 3200 29.6 / 27.6, 64 51.5 / 48.4, but 24 24.3 / 25.0; below, 8 of 8000 22.9 / 23.1, 32 of 1700
//     20.9 / 21.4, 16 13.9 / 15.5, 16 of 3200 18.1 / 19.3, two heads, 64 of 1700 14.1 / 15.1.  Rotated, whose pieces of approximated rows are cut well by the estimate, never: 64 of 3200 49.5 / 57.4, 24 of 3200 26.9 / 28.4, 16 of 8000
//     35.5 / 36.1, and at best (12 of 8000) 31.7 / 30.5.
constexpr bool worth_a_plan(int head_dim, bool turned, int per_cu, int batch, int n_kv_heads, int cap_retain, int n_approx) {
  if (batch < 2 || batch > kMaxPlanned || (head_dim == 64 && turned)) return false;
  const int64_t steps = ((int64_t)cap_retain + 127) / 128 + ((int64_t)n_approx + 127) / 128;
  return steps * batch * n_kv_heads >= (head_dim == 64 ? 6 : 3) * 256 * (int64_t)per_cu;
}

}  // namespace vec
