"""What the decode launches compute about rows, compiled for the host.  No GPU needed."""
import os
import subprocess

import pytest

from paper_2605_23258_amd import build

# every capacity, live length and block size; the step's own token (row cap where the block is full) and without it; every
# range of 128-row steps that a workgroup can have; every lane.  Prints the first entry outside the table, or that does not
# name the block of a row that has one.
PROGRAM = r"""
#include <cstdio>
#include "decode_rows.hpp"
int main() {
  for (int shift = 5; shift <= 8; ++shift)
    for (int cap = 1; cap <= 700; ++cap)
      for (int len = cap > 3 ? cap - 3 : 0; len <= cap + 1; ++len) {            // cap + 1: full, and the token
        const int entries = (cap - 1 >> shift) + 1;
        for (int begin = 0; begin < len; begin += 128)
          for (int end = begin + 128;; end += 128) {
            const int row_end = end < len ? end : len;
            for (int lane = 0; lane < 64; ++lane) {
              const int e = vec::block_entry(begin, row_end, cap, shift, lane), want = (begin >> shift) + lane;
              if (e < 0 || e >= entries || (want <= ((row_end < cap ? row_end : cap) - 1 >> shift) && e != want)) {
                printf("shift %d cap %d rows %d..%d lane %d: entry %d of %d\n", shift, cap, begin, row_end, lane, e, entries);
                return 1;
              }
            }
            if (end >= len) break;
          }
      }
  return 0;
}
"""


def run(tmp_path, program):
    (tmp_path / "rows.cpp").write_text(program)
    exe = str(tmp_path / "rows")
    subprocess.run([os.path.join(os.path.dirname(build.HIPCC), "amdclang++"), "-std=c++17", "-O2", "-w", "-I", build.CSRC,
                    str(tmp_path / "rows.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_block_table_entries_stay_in_the_table(tmp_path):
    run(tmp_path, PROGRAM)


# segments of every kind of length, few and many (sequence, head) pairs, both kinds of steps
SPLITS = r"""
#include <cstdio>
#include "decode_rows.hpp"
int main() {
  const int rows[] = {0, 1, 20, 100, 128, 129, 1000, 5000, 40000, 1000000, 2147483647};
  for (int kind = 0; kind < 72; ++kind) {
    const int group = kind / 4 % 3 == 0 ? 1 : kind / 4 % 3 == 1 ? 4 : 16;
    const vec::SplitCosts costs = vec::split_costs(kind & 1, kind & 2 ? 64 : 128, group, (vec::ApproxRows)(kind / 12 % 3), 1 + kind / 18);
    for (int pairs : {1, 2, 3, 8, 64, 300, 5000})
      for (int cap : rows)
        for (int n : rows) {
          int r = -1, a = -1;
          vec::pick_splits(costs, pairs, 1, cap, n, r, a);
          const bool none = cap == 0 && n == 0;
          if (r + a > vec::kMaxSplits || r < (cap > 0 || none) || a < (n > 0) || (cap == 0 && !none && r) || (n == 0 && a)) {
            printf("kind %d, %d pairs, %d and %d rows: %d + %d\n", kind, pairs, cap, n, r, a);
            return 1;
          }
        }
  }
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_splits_stay_within_their_number(tmp_path):
    """Every segment with rows gets a split, one without gets none, and both together get no more than a merge has room for."""
    run(tmp_path, SPLITS)


# A step's time was measured with the segments cut in every way: shape, and the cuts within 10 % of the best.  With the
# constants of bf16 and d = 128 for all kernels these took 1.1 to 1.8 times the best.
MEASURED = [
    # bf16, d, query heads per KV head, approximated rows plain (0), turned (1) or rebuilt (2), workgroups per CU, sequences, KV heads, capacity, approximated rows
    ((1, 64, 4, 0, 3, 24, 8, 1855, 1599), "5+3 3+2 4+3 5+4 2+2 5+5 6+4 6+5 7+4 3+3 4+5 6+3 4+6 3+4 5+6 2+3 7+5 7+3 4+4 4+2"),
    ((1, 64, 4, 0, 3, 16, 8, 1956, 1700), "2+2 2+4 3+3 4+2 7+5 5+4 3+2 2+3 7+6 3+4"),
    ((0, 128, 4, 0, 3, 32, 8, 665, 409), "1+1 2+1 3+3 1+2 4+3 2+3 3+2 3+4"),
    ((0, 128, 4, 0, 3, 8, 8, 665, 409), "6+6 7+5 5+3 4+4 5+6 5+5 4+3 6+5 3+4 3+3 6+4 4+5 7+4 5+4 8+7 8+4 7+7 9+3"),
    ((0, 64, 8, 0, 2, 6, 8, 665, 409), "5+5 3+2 4+4 6+4 4+6 2+3 2+2 4+5 5+4"),
    ((0, 128, 8, 0, 2, 6, 8, 665, 409), "5+5 6+4 5+4 4+4"),
    ((0, 64, 4, 1, 3, 18, 8, 317, 125), "1+2 3+2 2+2"),
    ((1, 128, 4, 2, 2, 16, 8, 3532, 3276), "2+2"),
    ((1, 128, 4, 2, 2, 1, 8, 1075, 819), "4+7 5+7 7+7 6+7 9+7"),
    ((1, 128, 8, 2, 2, 4, 8, 1894, 1638), "5+7 5+8 6+7 6+8 4+4"),
    ((1, 128, 4, 2, 2, 8, 8, 665, 409), "2+2 2+4 3+4 1+2"),
    ((1, 64, 4, 2, 2, 8, 8, 665, 409), "2+2 4+4 3+4 2+4 3+3"),
    # four workgroups fit a CU here, and the cuts for four were measured 8 to 25 % slower than these
    ((0, 128, 3, 0, 4, 16, 8, 1256, 1000), "3+3"), ((0, 128, 3, 0, 4, 24, 8, 1256, 1000), "2+2"), ((0, 128, 3, 0, 4, 8, 8, 1056, 200), "9+3"),
    ((0, 128, 3, 0, 4, 16, 8, 656, 400), "3+3"), ((0, 128, 3, 0, 4, 24, 8, 456, 800), "1+3"),
    # two, three and two, with registers that once let one, two and one fit
    ((0, 128, 10, 0, 2, 16, 8, 1256, 1000), "2+2"), ((0, 128, 5, 0, 3, 24, 8, 656, 400), "2+2"), ((0, 128, 10, 0, 2, 6, 8, 656, 400), "5+5"),
]


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_splits_are_among_the_fastest_measured(tmp_path):
    lines = "".join("  { int r, a; vec::pick_splits(vec::split_costs(%d, %d, %d, (vec::ApproxRows)%d, %d), %d, %d, %d, %d, r, a); char s[32]; sprintf(s, \" %%d+%%d \", r, a);"
                    " if (!strstr(\" %s \", s)) { printf(\"%s:%%s\\n\", s); bad = 1; } }\n" % (shape + (fast, shape)) for shape, fast in MEASURED)
    run(tmp_path, '#include <cstdio>\n#include <cstring>\n#include "decode_rows.hpp"\nint main() {\n  int bad = 0;\n' + lines + "  return bad;\n}\n")


# the same for the splits of one round
ONE_ROUND = r"""
#include <cstdio>
#include "decode_rows.hpp"
int main() {
  const int rows[] = {0, 1, 20, 128, 129, 1000, 5000, 40000, 1000000, 2147483647};
  for (int per_cu = 1; per_cu <= 4; ++per_cu)
    for (int pairs : {1, 2, 3, 8, 64, 100, 129, 257, 300, 383, 384, 5000})
      for (int least : {1, 2, 70})
        for (int cap : rows)
          for (int n : rows) {
            int r = -1, a = -1;
            const vec::SplitCosts costs = vec::split_costs(true, 128, 4, vec::ApproxRows::kPlain, per_cu);
            if (!vec::pick_one_round(costs, pairs, 1, cap, n, least, r, a)) continue;
            // one round, or one piece each and at least half a round more
            const long long at_once = 256 * per_cu, round = 4 * pairs >= 3 * at_once && r + a == 2 ? 2 * pairs : at_once;
            if (cap == 0 || n == 0 || r < least || r < 1 || a < 1 || r + a > vec::kMaxSplits || (long long)pairs * (r + a) > round ||
                r > (cap + 127ll) / 128 || a > (n + 127ll) / 128) {
              printf("%d per CU, %d pairs, %d and %d rows: %d + %d\n", per_cu, pairs, cap, n, r, a);
              return 1;
            }
          }
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_splits_of_one_round_make_one(tmp_path):
    run(tmp_path, ONE_ROUND)


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_a_plan_leaves_out_what_the_call_leaves_out(tmp_path):
    run(tmp_path, '#include "decode_rows.hpp"\nusing vec::planned_rows;\nint main() { return planned_rows(0, 500) || planned_rows(7, 500) != 500 || planned_rows(500, 0) || planned_rows(500, -3); }\n')


# Unequal sequences for which a plan and as many splits for every one were measured more than 3 % apart
PLANNED = [
    # head_dim, rotated keys, workgroups per CU, sequences, KV heads, largest capacity, most approximated rows, whether the plan is the faster
    (128, 0, 2, 2, 8, 1106, 850, 0), (128, 1, 2, 2, 8, 1106, 850, 0), (128, 0, 2, 3, 8, 1856, 1600, 0), (128, 1, 2, 4, 8, 1106, 850, 0),
    (128, 0, 2, 4, 2, 4256, 4000, 0), (128, 1, 2, 4, 2, 4256, 4000, 0), (128, 0, 2, 6, 2, 1106, 850, 0), (128, 1, 2, 8, 2, 4256, 4000, 0),
    (128, 0, 2, 8, 8, 1856, 1600, 1), (128, 1, 2, 6, 8, 4256, 4000, 1), (128, 0, 2, 16, 8, 1106, 850, 1), (128, 0, 2, 64, 2, 4256, 4000, 1),
    (128, 0, 2, 24, 8, 2999, 457, 1), (128, 1, 2, 24, 8, 2999, 457, 1), (128, 0, 2, 24, 8, 3456, 0, 1),
    (64, 0, 3, 3, 8, 4256, 4000, 0), (64, 0, 3, 16, 8, 1106, 850, 0), (64, 0, 3, 16, 8, 1856, 1600, 0), (64, 0, 3, 64, 2, 1106, 850, 0),
    (64, 1, 3, 64, 8, 1856, 1600, 0), (64, 1, 3, 24, 8, 1856, 1600, 0), (64, 1, 3, 6, 2, 4256, 4000, 0),
    (64, 0, 3, 10, 8, 4256, 4000, 1), (64, 0, 3, 12, 8, 4256, 4000, 1), (64, 0, 3, 28, 8, 1856, 1600, 1), (64, 0, 3, 32, 8, 1106, 850, 0), (64, 0, 3, 32, 8, 2256, 2000, 1), (64, 0, 3, 64, 8, 1856, 1600, 1),
    # one sequence, and more than a wave has lanes
    (128, 0, 2, 1, 8, 100000, 100000, 0), (128, 0, 2, 65, 8, 4000, 4000, 0),
]


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_plans_where_they_were_measured_faster(tmp_path):
    lines = "".join("  if (vec::worth_a_plan(%d, %d, %d, %d, %d, %d, %d) != %d) { printf(\"%s\\n\"); bad = 1; }\n" % (shape + (shape,)) for shape in PLANNED)
    run(tmp_path, '#include <cstdio>\n#include "decode_rows.hpp"\nint main() {\n  int bad = 0;\n' + lines + "  return bad;\n}\n")


# A plan's workgroups, one after another, over sequences of random and of extreme lengths: every granule belongs to one of them, no two
# partials share a place, a segment's lie next to each other from the one with granule 0 on, and there are no more than the merge has room for.
# The inverses a bit too small, exact and a bit too large.
PLAN = r"""
#include <cstdio>
#include <map>
#include <random>
#include <vector>
#include "decode_rows.hpp"
using namespace vec;
struct Segment { int n, next = 0, place = -1, count = 0, said_place = -1, said_count = 0; };
int check(const std::vector<int>& ret, const std::vector<int>& apx, int H, int per_cu, float plan_apx, float off) {
  const int B = (int)ret.size(), pairs = B * H, wgs = plan_workgroups(per_cu, pairs), most = plan_most_retained(per_cu, wgs);
  int log_rows = kLogGranule;
  std::vector<int> len[2];
  std::vector<Segment> segments[2];
  float top[2];
  for (;; ++log_rows) {
    for (int s = 0; s < 2; ++s) {
      len[s].clear(); segments[s].clear(); top[s] = 0.f;
      for (int b = 0; b < B; ++b) {
        int n = plan_granules(s ? apx[b] : ret[b], log_rows);
        if (s == 0 && apx[b] == 0 && n < 1) n = 1;
        len[s].push_back(plan_length(n));
        top[s] = std::max(top[s], (float)plan_length(n));
        for (int h = 0; h < H; ++h) { segments[s].push_back({}); segments[s].back().n = n; }
      }
    }
    if (!plan_too_long(std::max(top[0], top[1]), B, H, log_rows)) break;
  }
  long long total[2] = {0, 0};
  for (int s = 0; s < 2; ++s) for (int x : len[s]) total[s] += (long long)x * H;
  if (total[0] > kMaxPlanUnits * 1.0001 || total[1] > kMaxPlanUnits * 1.0001) { printf("line of %lld + %lld\n", total[0], total[1]); return 1; }
  auto inverse = [&](float x) { return 1.0f / x * off; };
  const int wgs_r = plan_retained(wgs, most, (int)total[0], (int)total[1], inverse((float)total[0] + (float)total[1] * plan_apx));
  if (wgs_r > wgs || (total[0] && wgs_r < 1) || (total[1] && wgs_r >= wgs)) { printf("%d of %d workgroups\n", wgs_r, wgs); return 1; }
  std::map<long long, int> places;
  for (int id = 0; id < wgs; ++id) {
    const int s = id >= wgs_r, mine = s ? id - wgs_r : id, share = plan_share((int)total[s], top[s], inverse((float)(s ? wgs - wgs_r : wgs_r)));
    const long long lo64 = (long long)mine * share;
    if (lo64 + share > 2147483647ll) { printf("share %d of workgroup %d\n", share, mine); return 1; }
    const int lo = (int)lo64;
    if (lo >= total[s]) continue;
    long long at = 0;
    int b = 0;
    while (at + (long long)len[s][b] * H <= lo) at += (long long)len[s][b++] * H;
    int h = plan_head(lo - (int)at, len[s][b], inverse((float)len[s][b]));
    at += (long long)h * len[s][b];
    if (h < 0 || h >= H || at > lo || at + len[s][b] <= lo) { printf("head %d\n", h); return 1; }
    while (b < B && at < lo64 + share) {
      Segment& g = segments[s][b * H + h];
      const PlanPiece piece = plan_piece((int)at, g.n, lo, share);
      if (piece.first < piece.last) {
        const int place = plan_place(id, b * H + h, s, pairs);
        if (piece.first != g.next || piece.last > g.n || place < 0 || place >= kMaxSplits * pairs || places.count(place)) {
          printf("segment %d of %d granules: %d..%d after %d, place %d\n", b * H + h, g.n, piece.first, piece.last, g.next, place);
          return 1;
        }
        places[place] = 1;
        if (g.count == 0) g.place = place;
        if (place != g.place + g.count) { printf("places %d and %d\n", g.place, place); return 1; }
        ++g.count;
        g.next = piece.last;
        if (piece.first == 0) { g.said_place = place; g.said_count = plan_partials((int)at, g.n, lo, share); }
      }
      at += plan_length(g.n);
      if (++h == H) { h = 0; ++b; }
    }
  }
  for (int s = 0; s < 2; ++s)
    for (const Segment& g : segments[s])
      if (g.next != g.n || g.count > kMaxSplits / 2 || g.count != g.said_count || (g.n && g.place != g.said_place)) {
        printf("segment of %d granules: %d, %d partials at %d, said %d at %d\n", g.n, g.next, g.count, g.place, g.said_count, g.said_place);
        return 1;
      }
  return 0;
}
int main() {
  std::mt19937 rng(1);
  const float offs[] = {1.f - 1.2e-7f, 1.f, 1.f + 1.2e-7f};
  for (int i = 0; i < 30000; ++i) {
    const int B = 2 + rng() % (i % 5 ? 20 : 63), H = i % 7 ? 1 + rng() % 8 : 1 + rng() % 40, per_cu = 1 + rng() % 4;
    // of one case the lengths reach from up to a few granules to up to all that 32 bits hold
    auto length = [&](int bits) { return rng() % 4 == 0 ? 0 : (int)(rng() >> (31 - (bits ? rng() % bits : 0)) & 0x7fffffff) + (int)(rng() % 2); };
    const int bits_r = 1 + rng() % (i % 10 ? 17 : 30), bits_a = 1 + rng() % (i % 10 ? 17 : 30);
    std::vector<int> ret, apx;
    for (int b = 0; b < B; ++b) { ret.push_back(length(bits_r)); apx.push_back(i % 11 ? length(bits_a) : 0); }
    if (i % 13 == 0) ret.assign(B, ret[0]), apx.assign(B, apx[0]);
    if (i % 17 == 0) ret.assign(B, 0);
    if (check(ret, apx, H, per_cu, i % 2 ? 1.f : kPlanTurned, offs[i % 3])) { printf("case %d: %d sequences, %d heads\n", i, B, H); return 1; }
  }
  // the longest lines
  for (int B : {2, 64}) for (int H : {1, 8, 1000}) for (int n : {2147483646, 1 << 30, 1 << 20})
    if (check(std::vector<int>(B, n), std::vector<int>(B, n / 3), H, 2, 1.f, 1.f)) { printf("%d sequences of %d, %d heads\n", B, n, H); return 1; }
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_plans_share_every_row_out_once(tmp_path):
    run(tmp_path, PLAN)


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_every_cu_of_a_plan_keeps_a_workgroup_for_approximated_rows(tmp_path):
    """Of the workgroups of a CU, 256 apart, all but the last are for retained rows where these are nearly all of the work (64 dims, three per
    CU: half of all, as with two, took up to 8 % longer); with less of them the work says how many, but no
    more than half up to three fifths of the work."""
    run(tmp_path, '#include "decode_rows.hpp"\nint main() {\n  for (int per_cu = 2; per_cu <= 4; ++per_cu) {\n    const int wgs = vec::plan_workgroups(per_cu, 200);\n'
        '    const int most = vec::plan_most_retained(per_cu, wgs);\n'
        '    if (wgs != 256 * per_cu || most != 256 * (per_cu - 1) || vec::plan_retained(wgs, most, 100000, 100, 1.f / 100100.f) != most) return 1;\n'
        '    if (vec::plan_retained(wgs, most, 1010, 1000, 1.f / 2010.f) != wgs / 2) return 1;\n'
        '    if (vec::plan_retained(wgs, most, 1000, 3000, 1.f / 4000.f) != wgs / 4 || vec::plan_retained(wgs, most, 1000, 0, 1.f / 1000.f) != wgs) return 1;\n  }\n  return 0;\n}\n')


# Plain rows of 128 dims whose cuts were measured both ways, more than 2 % apart: sequences (eight heads, two workgroups per CU), capacity,
# approximated rows; the cut in one round's order, or nothing where the estimate's was the faster
ONE_ROUND_MEASURED = [
    ((33, 2256, 2000), ""), ((40, 2256, 2000), ""), ((36, 956, 700), ""), ((36, 1456, 2400), ""), ((36, 2656, 1200), ""), ((48, 2656, 1200), ""), ((64, 2656, 1200), ""),
    ((48, 2256, 2000), "1+1"), ((96, 2256, 2000), "1+1"), ((52, 956, 700), "1+1"), ((128, 956, 700), "1+1"), ((48, 1456, 2400), "1+1"), ((80, 1456, 2400), "1+1"),
    ((22, 1856, 3500), ""), ((28, 1856, 3500), ""), ((31, 1856, 3500), ""), ((28, 1256, 3000), ""), ((24, 1256, 3000), "1+1"), ((21, 1856, 3500), "1+2"), ((17, 1256, 3000), "1+2"),
    ((24, 2256, 2000), "1+1"), ((32, 2256, 2000), "1+1"), ((17, 956, 700), "2+1"), ((32, 956, 700), "1+1"), ((26, 2656, 1200), "1+1"), ((17, 2656, 1200), "2+1"),
    ((16, 3532, 3276), "2+2"), ((30, 3256, 1000), ""),
]


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_one_round_where_it_was_measured_faster(tmp_path):
    lines = "".join("  { int r = 0, a = 0; char s[32] = \"\"; if (vec::pick_one_round(vec::split_costs(true, 128, 4, vec::ApproxRows::kPlain, 2), %d, 8, %d, %d, 1, r, a)) sprintf(s, \"%%d+%%d\", r, a);"
                    " if (strcmp(s, \"%s\")) { printf(\"%s: %%s\\n\", s); bad = 1; } }\n" % (shape + (cut, shape)) for shape, cut in ONE_ROUND_MEASURED)
    run(tmp_path, '#include <cstdio>\n#include <cstring>\n#include "decode_rows.hpp"\nint main() {\n  int bad = 0;\n' + lines + "  return bad;\n}\n")
