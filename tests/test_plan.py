"""How launches are cut into workgroups, compiled for the host.  No GPU needed."""
import subprocess

from paper_2605_23258_amd import build

# Every mix of three prompts' units (in strides), with heads that fit the CUs many times over, once, and not at all: the fewest
# units per part that fit, or the longest prompt's; found in six looks, however many steps there are.
PROGRAM = r"""
#include <cstdio>
#include "plan.hpp"
int main() {
  for (int heads : {1, 2, 3, 8, 40, 64, 85, 86, 128, 300})
    for (int a = 1; a <= 64; ++a)
      for (int b = 1; b <= 64; b += 7)
        for (int c = 1; c <= 64; c += 9) {
          const int n[3] = {a, b, c}, most = std::max(a, std::max(b, c));
          int looks = 0;
          auto workgroups = [&](int64_t step) {
            ++looks;
            int64_t parts = 0;
            for (int x : n) parts += (x + step - 1) / step;
            return parts * heads;
          };
          int want = 1;
          while (want < most && workgroups(want) > 256) ++want;
          looks = 0;
          const int found = (int)vec::smallest_step(most, 256, workgroups), got = vec::part_units(n, 3, heads);
          if (found != want || got != want || looks > 6) {
            printf("heads %d units %d %d %d: steps %d, %d after %d looks, not %d\n", heads, a, b, c, found, got, looks, want);
            return 1;
          }
        }
  return 0;
}
"""


def test_units_per_part(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
