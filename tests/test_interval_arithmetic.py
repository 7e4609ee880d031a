"""The dK/dV loop's element mask on bounds over the whole int32 range: the functions that the kernel uses, compiled for
the host with the undefined-behaviour sanitizer (a signed overflow ends the program) and compared with 64-bit arithmetic."""
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
  std::vector<int> bounds = {INT_MIN, INT_MIN + 1, INT_MIN + 130, -131, -1, 0, 1, 63, 64, 65, 4096, 131071, 1 << 30,
                             INT_MAX - 130, INT_MAX - 1, INT_MAX};
  std::mt19937 gen(7);
  std::uniform_int_distribution<int> any(INT_MIN, INT_MAX);
  for (int k = 0; k < 24; ++k) bounds.push_back(any(gen));
  std::vector<int> rows = {0, 1, 28, 60, 64, 4092, 131040, (1 << 30) - 32};   // first row of a block's registers
  long long checked = 0;
  for (int start : bounds)
    for (int end : bounds)
      for (int row : rows) {
        const unsigned length = interval_length(start, end), offset = interval_offset(row, start);
        for (unsigned dr = 0; dr < 28; ++dr, ++checked) {
          const long long r = (long long)row + dr;
          if (in_interval(offset + dr, length) != (start <= r && r < end)) {
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
    source, program = tmp_path / "interval.cpp", tmp_path / "interval"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, str(source),
                    "-o", str(program)], check=True, timeout=120)
    done = subprocess.run([str(program)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout + done.stderr
    assert done.stdout.startswith("checked")


def test_the_kernel_forms_offsets_and_lengths_with_them():
    """No other arithmetic on the bounds in the dK/dV loop."""
    with open(os.path.join(CSRC, "fm_bwd.hip")) as f:
        text = f.read()
    for name in ("interval_length(b_lts, b_lte)", "interval_length(b_uts, b_ute)", "interval_offset(row, s_a)",
                 "interval_offset(row, s_b)"):
        assert name in text, name
    for bound in ("s_a", "s_b", "b_lts", "b_lte", "b_uts", "b_ute"):
        assert f"- {bound}" not in text and f"{bound} -" not in text, bound
