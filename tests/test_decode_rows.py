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
  for (int step : {32, 64, 128})
    for (int pairs : {1, 2, 3, 8, 64, 300, 5000})
      for (double apx : {1.0, 2.2})
        for (int cap : rows)
          for (int n : rows) {
            int r = -1, a = -1;
            vec::pick_splits(step, pairs, 1, cap, n, apx, r, a);
            const bool none = cap == 0 && n == 0;
            if (r + a > vec::kMaxSplits || r < (cap > 0 || none) || a < (n > 0) || (cap == 0 && !none && r) || (n == 0 && a)) {
              printf("steps of %d, %d pairs, %d and %d rows: %d + %d\n", step, pairs, cap, n, r, a);
              return 1;
            }
          }
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the ROCm toolchain")
def test_splits_stay_within_their_number(tmp_path):
    """Every segment with rows gets a split, one without gets none, and both together get no more than a merge has room for."""
    run(tmp_path, SPLITS)
