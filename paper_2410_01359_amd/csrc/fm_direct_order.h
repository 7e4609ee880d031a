// Which unit a workgroup of a launch over direct units takes (see fm_common.h).  Plain integer code: the host compiles it
// too.
#pragma once
#include "fm_interval.h"

// Workgroup x runs on XCD x % 8, and each XCD has an L2 of its own.  The slices (batch row and K/V head; `group` query heads of
// it take turns) are dealt to m classes of XCDs in contiguous runs, m = the largest power of two up to 8 that divides their
// count, so that a slice is worked on by at most 8 / m XCDs and the bounds of its batch row are read by as few.  An XCD takes its
// slices' blocks in step, in the order 0, 1, 2, ...: what is longest in masks with a causal side comes first for all of them
// (the callers count row blocks from the last).
//  - Slices of at least four blocks to each XCD of their class are shared by all of it: its XCDs take chunks of up to eight
//    neighbouring blocks in turn, back and forth, so that they get equal shares of a length that falls from block to block;
//    neighbours have much of their tiles in common, a window's nearly all.  Where the turns do not come out even, each slice
//    begins one XCD further on than the one before, so that what is over does not go to the same XCDs for all of them.
//  - Shorter ones would leave XCDs without a block, and every XCD would fetch every slice: each XCD has as many of them to
//    itself as there are for all, and the fewer than 8 / m left over are shared block by block, ahead of the others.
// An XCD then has at most one block (chunk) of a group more than its even share, whatever the counts.  With all slices shared
// and begun at the same XCD, the XCDs past the last block had nothing: one XCD all 255 units of as many slices of one block.
// Forward / backward in us, causal, all begun at one XCD -> now:
//   d = 128  255 slices, N = 128  70.5 / 177 -> 11.3 / 30;  three rows of 25, N = 512  31.8 / 93 -> 16.4 / 46
//   d = 64   255 slices, N = 128  23.3 / 55 -> 7.2 / 17;    three rows of 25, N = 512  19.4 / 52 -> 11.8 / 29
// With short slices shared block by block, too, 85 of 384 tokens took 1.16 / 1.08 and 75 of 1024 1.10 / 1.05 times as long
// (d = 128); with those of 16 and more blocks whole, 20 of 4000 (d = 64) 1.06 / 1.03.
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
  int own;                              // slices of a class
  int classes, sharing, chunk;          // m, XCDs of a class, blocks taken together: powers of two, as their logarithms
  int whole;                            // short slices: those that an XCD has to itself; -1: its class shares all
  int turns;                            // of an XCD, a chunk each: at every slice, or of short ones at those shared together
  int turned;                           // whether a slice begins one XCD further on than the one before
};
FM_HOST_DEVICE inline FmDirectOrder fm_direct_order(int slices, int blocks) {
  constexpr int kLogXcds = 3, kLogTurns = 2, kLogChunk = 3;
  FmDirectOrder o = {slices, 0, kLogXcds, 0, -1, 0, 0};
  for (; o.classes < kLogXcds && o.own % 2 == 0; o.own /= 2, --o.sharing) ++o.classes;
  int chunks;
  if (o.sharing == 0 || blocks >> (kLogTurns + o.sharing) == 0) {
    o.whole = o.own >> o.sharing;
    chunks = blocks * (o.own & ((1 << o.sharing) - 1));
  } else {
    while (o.chunk < kLogChunk && blocks >> (o.chunk + 1 + kLogTurns + o.sharing)) ++o.chunk;
    chunks = (blocks + (1 << o.chunk) - 1) >> o.chunk;
    o.turned = blocks % (2 << (o.sharing + o.chunk)) != 0;
  }
  o.turns = (chunks + (1 << o.sharing) - 1) >> o.sharing;
  return o;
}
// Workgroups of the launch.
FM_HOST_DEVICE inline int fm_direct_grid(const FmDirectOrder& o, int group, int blocks) {
  return 8 * group * (o.whole < 0 ? o.own * (o.turns << o.chunk) : o.turns + o.whole * blocks);
}
// The slice, member of its group and block that workgroup x takes; block = -1: none.
struct FmDirectUnit {
  int slice, member, block;
};
FM_HOST_DEVICE inline FmDirectUnit fm_direct_unit(const FmDirectOrder& o, int x, int group, int blocks) {
  const int xcd = x & 7, p = xcd >> o.classes, last = (1 << o.sharing) - 1;
  int at = x >> 3, slice, member, block;   // at: which of the XCD's workgroups, slice: of the class
  const int ahead = o.whole < 0 ? 0 : o.turns * group;
  if (at < ahead) {   // short slices that the class shares: block 0 of all, block 1, ..., the XCDs in turn
    const int turn = group == 1 ? at : at / group, n = o.own & last, pass = n == 1 ? turn : turn / n;
    const int k = (turn << o.sharing) + (pass & 1 ? last - p : p);
    member = at - turn * group;
    block = n == 1 ? k : k / n;
    slice = (o.whole << o.sharing) + k - block * n;
  } else {
    at -= ahead;
    const int n = o.whole < 0 ? o.own : o.whole, step = n == 1 ? at : at / n, i = group == 1 ? step : step / group;
    slice = at - step * n;
    member = step - i * group;
    block = i;
    if (o.whole < 0) {
      const int turn = i >> o.chunk, mine = (p + (o.turned ? slice : 0)) & last;
      block = (((turn << o.sharing) + (turn & 1 ? last - mine : mine)) << o.chunk) + (i & ((1 << o.chunk) - 1));
    } else {
      slice += p * n;
    }
  }
  return FmDirectUnit{(xcd & ((1 << o.classes) - 1)) * o.own + slice, member, block < blocks ? block : -1};
}
