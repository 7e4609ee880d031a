"""The dK/dV loop's element mask, 32 rows in a word, over the whole int32 range: the function that the kernel uses, compiled
for the host with the undefined-behaviour sanitizer and compared with 64-bit arithmetic row by row."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_01359_amd", "csrc")

PROGRAM = r"""
#include <climits>
#include <cstdio>
#include <random>
#include <vector>
#include "fm_interval.h"

int main() {
  std::vector<int> bounds = {INT_MIN, INT_MIN + 1, INT_MIN + 130, -131, -1, 0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 4096,
                             131071, 1 << 30, (1 << 30) + 7, INT_MAX - 130, INT_MAX - 31, INT_MAX - 1, INT_MAX};
  std::mt19937 gen(7);
  std::uniform_int_distribution<int> any(INT_MIN, INT_MAX);
  for (int k = 0; k < 24; ++k) bounds.push_back(any(gen));
  std::vector<int> rows = {0, 4, 32, 36, 64, 4092, 131040, (1 << 30) - 32, INT_MAX - 31};   // first row of a block
  long long checked = 0;
  for (int start : bounds)
    for (int end : bounds)
      for (int row : rows) {
        const unsigned bits = interval_rows(interval_offset(row, start), interval_length(start, end));
        for (int p = 0; p < 32; ++p, ++checked) {
          const long long r = (long long)row + p;
          if (((bits >> p) & 1u) != (unsigned)(start <= r && r < end)) {
            std::printf("[%d, %d) row %lld\n", start, end, r);
            return 1;
          }
        }
      }
  std::printf("checked %lld\n", checked);
  return 0;
}
"""


def test_every_int32_bound(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    source, program = tmp_path / "rows.cpp", tmp_path / "rows"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, str(source),
                    "-o", str(program)], check=True, timeout=120)
    done = subprocess.run([str(program)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout + done.stderr
    assert done.stdout.startswith("checked")
