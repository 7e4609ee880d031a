"""The LDS layout of a tile, compiled for the host: every 16-byte chunk has a place of its own, each lane of a copy reads the row
and column that its place in LDS stands for (row strides up to the limit of the strided entry points), a further column is where
add_col says, and the operand reads of both matrix shapes and the transpose reads meet no bank twice in a clock."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_01359_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <set>
#include <vector>
#include "fm_tile_layout.h"

// lanes that a 128-bit read serves in the same clock: 16 of each half of the wave
static const int kClock[2][16] = {{0, 1, 2, 3, 12, 13, 14, 15, 20, 21, 22, 23, 24, 25, 26, 27},
                                  {4, 5, 6, 7, 8, 9, 10, 11, 16, 17, 18, 19, 28, 29, 30, 31}};

template <int D>
int check() {
  using L = TileLayout<D>;
  std::set<int> places;
  for (int row = 0; row < 64; ++row)
    for (int col = 0; col < L::RS; ++col) {
      const int at = L::off(row, col);
      if (at % 16 != col % 16 || L::off(row, col & ~15) != (at & ~15)) return 1;
      if (at < 0 || at >= 64 * L::RS || L::off(row % 16, col) + row / 16 * 16 * L::RS != at) return 2;
      places.insert(at);
      for (int colc = 0; colc + col < L::RS; colc += 32)
        if ((col < 32 || (colc % 64 == 0 && col < 64)) && (int)L::add_col(at, colc) != L::off(row, col + colc)) return 3;
    }
  if ((int)places.size() != 64 * L::RS) return 4;

  std::vector<long long> strides = {L::RS, 3 * L::RS, 2 * 12345 * 8, 2 * ((1 << 24) - 8)};
  for (long long grs : strides)
    for (int wave = 0; wave < 4; ++wave)
      for (int lane = 0; lane < 64; ++lane) {
        CopyLanes<D> lanes;
        lanes.init(lane, (int)grs);
        const char* const slice = (const char*)(1ll << 40);
        for (int s = 0; s < CopyLanes<D>::NINST; ++s) {
          const long long from = CopyLanes<D>::wave_base(slice, wave, (int)grs) + lanes.v[s] + s * 1024 - slice;
          const int row = wave * 16 + lane / 4, to = wave * 16 * L::RS + s * 1024 + 16 * lane;
          const long long col = from - row * grs;
          if (col < 0 || col >= L::RS || L::off(row, (int)col) != to || col != CopyLanes<D>::source_col(lane, s)) return 5;
        }
      }

  for (int half = 0; half < 2; ++half)
    for (const auto& clock : kClock)
      for (int kk = 0; kk < L::RS / 32; ++kk) {
        std::set<int> rows32, rows16;
        for (int lane : clock) {
          const int l = half * 32 + lane;
          rows32.insert(L::off(l % 32, 16 * (l / 32) + 32 * kk) / 16 % 16);
          if (kk < L::PANELS) rows16.insert(L::off(l % 16, 16 * (l / 16) + 64 * kk) / 16 % 16);
        }
        if (rows32.size() != 16 || (kk < L::PANELS && rows16.size() != 16)) return 6;
      }
  for (int half = 0; half < 2; ++half)
    for (int n = 0; n < L::RS / 32; ++n)
      for (int hi = 0; hi < 2; ++hi) {
        std::set<int> of32, of16;
        for (int lane = 0; lane < 32; ++lane) {
          const int l = half * 32 + lane, i = l & 15;
          if (n < L::PANELS) of32.insert(L::off(4 * (l / 32) + (i >> 2) + 8 * hi, (16 * ((l >> 4) & 1) + 4 * (i & 3)) * 2 + 64 * n) / 8 % 32);
          of16.insert(L::off(4 * (l / 16) + (i >> 2), 8 * (i & 3) + 32 * n) / 8 % 32);
        }
        if ((n < L::PANELS && of32.size() != 32) || of16.size() != 32) return 7;
      }
  return 0;
}

int main() {
  const int a = check<64>(), b = check<128>();
  std::printf("%d %d\n", a, b);
  return a || b;
}
"""


def test_layout_copies_and_banks(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    source, program = tmp_path / "layout.cpp", tmp_path / "layout"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wno-unknown-pragmas", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", CSRC, str(source), "-o", str(program)], check=True, timeout=120)
    done = subprocess.run([str(program)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout + done.stderr
