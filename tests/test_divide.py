"""The division by a host-made reciprocal (csrc/divide.h) over the ranges that the score passes use it for."""
import os
import subprocess

from paper_2604_10235_amd import build

# every (workgroup, what the even shares leave) of launches of up to 2048 teams; the ends of the quotients' steps and both sides of
# them for every divisor that a quotient below 65536 (layers * heads) allows in a sequence of 2^30 positions
CHECK = r"""
#include <cstdio>
#include "divide.h"
using namespace codecomp;
int main() {
  for (int d = 1; d <= 2048; d += d < 300 ? 1 : 7)
    for (int g = 0; g <= d; ++g)
      for (int left = 0; left < d; left += left < 40 || left > d - 40 ? 1 : 37)
        if (divide(g * left, d, 1.0f / (float)d) != g * left / d) return 1;
  for (long d = 1; d < (1l << 30); d += 1 + d / 50)
    for (long q = 0; q < 65536 && q * d < (1l << 30); q += 1 + q / 20)
      for (long x = q * d - 2; x <= q * d + 2; ++x)
        if (x >= 0 && x < (1l << 30) && divide((int)x, (int)d, 1.0f / (float)d) != (int)(x / d)) return 2;
  return 0;
}
"""


def test_divide(tmp_path):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(CHECK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(build.ROCM, "include"), "-I", build.CSRC,
                    str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
