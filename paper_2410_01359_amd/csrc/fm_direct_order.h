// Which unit a workgroup of a launch over direct units takes (see fm_common.h).  Plain integer code: the host compiles it
// too.
#pragma once
#include "fm_interval.h"

// Workgroup x runs on XCD x % 8, and each XCD has an L2 of its own.  The slices (batch row and K/V head; `group` query heads of
// it take turns) are dealt to m classes of XCDs in contiguous runs, m = the largest power of two up to 8 that divides their
// count, so that a slice is worked on by 8 / m XCDs (one where the slices fill rounds of eight) and the bounds of its batch row are read by as few.
// An XCD takes its slices' blocks in step, in the order 0, 1, 2, ...: what is longest in masks with a causal side comes first
// for all of them (the callers count row blocks from the last).  XCDs that share a slice take chunks of up to eight
// neighbouring blocks in turn, back and forth, so that they get equal shares of a length that falls from block to block; four
// turns at least.  Neighbours have much of their tiles in common, a window's nearly all.
//
// Before, an XCD had one contiguous run of units, slice after slice: of few heads one XCD had all the long units of a causal mask
// and another all the short ones; in several rounds, units started in the order of the slices; and where two workgroups share a
// compute unit, they were equally long.  Loop times in us, before -> now (fwd / dQ / dK,dV):
//   d = 128  2 heads, N = 16384   causal 240 -> 211 / 304 -> 280 / 377 -> 246, documents of 700 tokens 64 -> 63 / 76 -> 75 / 79 -> 64
//            3 heads, N = 8192    causal 112 -> 108 / 147 / 158 -> 111;  16 heads, N = 2048 (one round, a unit to a compute unit) as before
//            32 heads on 8 K/V heads, two rows of 2048, shared questions   dK/dV 122 -> 112
//   d = 64   16 heads, N = 2048   causal 28.8 -> 23.5 / 34.7 -> 28.9 / 33.8 -> 28.4, documents 37 -> 31 / 38 -> 37 / 42 -> 40
//            2 heads, N = 16384   causal 165 -> 133 / 194 -> 161 / 218 -> 162;  4 heads, N = 8192, documents 40 -> 41 / 46 -> 47 / 37 -> 36
// Windows of 256 keep their times within 2 to 3 %.  With the blocks of a slice dealt to its XCDs one by one, windows took up to 8 %
// longer (each tile came to every L2) and the three heads' documents 46 instead of 55 us of dK/dV.
struct FmDirectOrder {
  int own;                              // slices of an XCD
  int classes, sharing, chunk;          // m, XCDs of a slice, blocks taken together: powers of two, as their logarithms
};
FM_HOST_DEVICE inline FmDirectOrder fm_direct_order(int slices, int blocks) {
  constexpr int kLogXcds = 3, kLogTurns = 2, kLogChunk = 3;
  FmDirectOrder o = {slices, 0, kLogXcds, 0};
  for (; o.classes < kLogXcds && o.own % 2 == 0; o.own /= 2, --o.sharing) ++o.classes;
  if (o.sharing)
    while (o.chunk < kLogChunk && blocks >> (o.chunk + 1 + kLogTurns + o.sharing)) ++o.chunk;
  return o;
}
// Workgroups of the launch.
FM_HOST_DEVICE inline int fm_direct_grid(const FmDirectOrder& o, int group, int blocks) {
  const int round = 1 << (o.sharing + o.chunk);
  return 8 * o.own * group * ((blocks + round - 1) / round << o.chunk);
}
// The slice, member of its group and block that workgroup x takes; block = -1: none.
struct FmDirectUnit {
  int slice, member, block;
};
FM_HOST_DEVICE inline FmDirectUnit fm_direct_unit(const FmDirectOrder& o, int x, int group, int blocks) {
  const int xcd = x & 7, turn = (x >> 3) / o.own, j = group == 1 ? turn : turn / group;
  const int chunk = j >> o.chunk, mine = (xcd >> o.classes) ^ (chunk & 1 ? (1 << o.sharing) - 1 : 0);
  const int block = (((chunk << o.sharing) + mine) << o.chunk) + (j & ((1 << o.chunk) - 1));
  return FmDirectUnit{(xcd & ((1 << o.classes) - 1)) * o.own + (x >> 3) - turn * o.own, turn - j * group,
                      block < blocks ? block : -1};
}
