"""The order of direct units: every unit is taken by exactly one workgroup of the launch, the workgroups beyond take none, an
XCD (workgroup number modulo 8) works on the run of slices of its class, a slice's blocks all go to one XCD (as many slices to each)
or in equal shares to the class, each XCD gets its share of all units, rounded up, and of a causal mask's work, and the launch
holds no more workgroups than that."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_01359_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <set>
#include <vector>
#include "fm_direct_order.h"

int main() {
  long long checked = 0;
  for (int n = 1; n < 5000; ++n)
    for (long long x : {0ll, 1ll, n - 1ll, 1ll * n, n + 1ll, 1000ll * n - 1, 1000ll * n, 0x7fffffffll / n * n - 1, 0x7fffffffll / n * n, 0x7fffffffll})
      if (const FmDivisor d = fm_divisor(n); fm_div((int)x, d) != x / n) {
        std::printf("%lld / %d is not %d\n", x, n, fm_div((int)x, d));
        return 1;
      }
  for (int slices : {1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 20, 24, 25, 32, 40, 64, 75, 100, 125, 127, 150, 175, 250, 252, 255})
    for (int group : {1, 2, 3, 4, 5, 8})
      for (int blocks : {1, 2, 3, 4, 5, 6, 7, 8, 9, 16, 31, 32, 33, 63, 64, 65, 84, 127, 128, 129, 255, 256, 257, 1024})
      for (bool at_once : {false, true}) {
        const FmDirectOrder o = fm_direct_order(slices, group, blocks, at_once);
        const int grid = fm_direct_grid(o), classes = 1 << o.classes;
        const int whole = o.deal == FM_DEAL_WHOLE ? o.own * classes / 8 : 0;   // slices that an XCD has to itself
        std::vector<int> taken(slices * group * blocks);
        std::vector<std::vector<int>> share(8, std::vector<int>(slices));   // blocks of a slice that an XCD works on
        std::vector<long long> units(8), work(8);   // of an XCD; a causal mask's block 0 is the longest
        for (int x = 0; x < grid; ++x, ++checked) {
          const FmDirectUnit u = group == 1 ? fm_direct_unit<false>(o, x) : fm_direct_unit<true>(o, x);
          if (u.block < 0) continue;
          if (u.slice < 0 || u.slice >= slices || u.member < 0 || u.member >= group || u.block >= blocks ||
              u.slice / o.own != x % 8 % classes) {
            std::printf("%d %d %d: workgroup %d takes %d %d %d\n", slices, group, blocks, x, u.slice, u.member, u.block);
            return 1;
          }
          ++taken[(u.slice * group + u.member) * blocks + u.block];
          ++share[x % 8][u.slice];
          ++units[x % 8];
          work[x % 8] += blocks - u.block;
        }
        for (int n : taken)
          if (n != 1) {
            std::printf("%d %d %d: a unit is taken %d times\n", slices, group, blocks, n);
            return 1;
          }
        std::vector<int> alone(8);
        for (int s = 0; s < slices; ++s)
          if (o.deal == FM_DEAL_RUNS) {
            ;
          } else if (8 / classes * whole > s % o.own) {
            for (int a = 0; a < 8; ++a) alone[a] += share[a][s] == group * blocks;
          } else {
            for (int a = 0; a < 8; ++a)
              for (int b = 0; b < 8; ++b)
                if (a % classes == s / o.own && b % classes == s / o.own &&
                    share[a][s] - share[b][s] > group << o.chunk) {
                  std::printf("%d %d %d: slice %d is shared %d : %d\n", slices, group, blocks, s, share[a][s], share[b][s]);
                  return 1;
                }
          }
        for (int a = 0; a < 8; ++a)
          if (alone[a] != whole) {
            std::printf("%d %d %d: XCD %d has %d slices to itself\n", slices, group, blocks, a, alone[a]);
            return 1;
          }
        if (o.deal == FM_DEAL_RUNS)
          for (int a = 0; a < 8; ++a) {   // a run of the class's units: of at most one slice more than the even share, rounded up
            int touched = 0;
            for (int s = 0; s < slices; ++s) touched += share[a][s] > 0;
            if (!at_once || touched > (o.own * classes + 7) / 8 + 1) {
              std::printf("%d %d %d: XCD %d works on %d slices\n", slices, group, blocks, a, touched);
              return 1;
            }
          }
        // An XCD has no unit more than its even share, and of the work a chunk of the longest more at most.
        const long long all = 1ll * slices * group * blocks, even = (all + 7) / 8;
        for (int x = 0; x < 8; ++x)
          if (units[x] > even || (o.deal != FM_DEAL_RUNS && 8 * work[x] > all * (blocks + 1) / 2 + 8ll * (group << o.chunk) * blocks)) {
            std::printf("%d %d %d: XCD %d has %lld of %lld units, work %lld\n", slices, group, blocks, x, units[x], all, work[x]);
            return 1;
          }
        if (grid != 8 * even) {
          std::printf("%d %d %d: grid %d\n", slices, group, blocks, grid);
          return 1;
        }
      }
  std::printf("checked %lld\n", checked);
  return 0;
}
"""


def test_every_unit_is_taken_once(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    source, program = tmp_path / "order.cpp", tmp_path / "order"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, str(source),
                    "-o", str(program)], check=True, timeout=120)
    done = subprocess.run([str(program)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout + done.stderr
    assert done.stdout.startswith("checked")
