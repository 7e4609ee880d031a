// Which unit a workgroup of a launch over direct units takes (see fm_common.h).  Plain integer code: the host compiles it
// too.
#pragma once
#include "fm_interval.h"

// Workgroup x runs on XCD x % 8, and each XCD has an L2 of its own.  The slices (batch row and K/V head; `group` query heads of
// it take turns) are dealt to m classes of XCDs in contiguous runs, m = the largest power of two up to 8 that divides their
// count, so that a slice is worked on by at most 8 / m XCDs and the bounds of its batch row are read by as few.  Every XCD of a
// class gets as many units, to one: where units are about as many as compute units, an XCD with one too many takes twice as long.
// An XCD takes its slices' blocks in step, in the order 0, 1, 2, ...: what is longest in masks with a causal side comes first
// for all of them (the callers count row blocks from the last).
//  - Turns, for slices of at least four blocks to each XCD of their class: its XCDs take chunks of up to eight neighbouring
//    blocks in turn, back and forth, so that they get equal shares of a length that falls from block to block; neighbours
//    have much of their tiles in common, a window's nearly all.  With an odd number of turns each slice begins one XCD further
//    on than the one before.  The blocks after the last whole turn go round one by one, slice after slice.
//  - Whole, for shorter slices, of which XCDs would be left without a block or every XCD would fetch every one: each XCD has
//    as many of them to itself as there are for all, and the blocks of the fewer than 8 / m others go round one by one, spread
//    evenly among those, so that the longest of both come first.
//  - Runs, where each compute unit has one unit at most, so that no order matters, and turns would bring several slices to
//    every XCD of a class: each has a contiguous run of units.
// Forward / backward in us, causal (3 slices: window 256), all slices in turns that begin at the same XCD -> now:
//   255 slices, N = 128          d = 128  70.5 / 177 -> 11.2 / 30   d = 64  23.3 / 55 -> 7.2 / 17    one XCD had all 255 units
//   three rows of 25, N = 512    d = 128  31.8 / 93 -> 16.4 / 46    d = 64  19.4 / 52 -> 11.8 / 29   four XCDs had none
//   3 slices, N = 5376           d = 128  21.4 / 48 -> 13.1 / 30                                  an XCD had 36 units for 32 compute units
//   7 slices, N = 1920           d = 128  25.1 / 62 -> 24.3 / 59                                  every XCD fetched every slice
// Against turns, runs take 1 % longer where a class has a single slice (1 of 8192 tokens, 4 of 1000), and with two units to
// a compute unit 1.2 times as long (12 of 2048, d = 64).  With short slices in turns, too, 85 of 384 tokens took 1.16 /
// 1.08 and 75 of 1024 1.10 / 1.05 times as long (d = 128); with those of 16 and more blocks whole, 20 of 4000 (d = 64) 1.06 / 1.03.
// With the blocks of the others ahead of the whole slices instead of among them, three rows of 10 heads on 5 took 1.04 / 1.03 (1792
// tokens, d = 128) and 1.08 / 1.05 (967, d = 64), 75 of 1024 0.96 / 0.97 times as long; behind them 1.1 to 1.2 throughout.
//
// Before turns, an XCD had one contiguous run of units, slice after slice: of few heads one XCD had all the long units of a causal mask
// and another all the short ones; in several rounds, units started in the order of the slices; and where two workgroups share a
// compute unit, they were equally long.  Loop times in us, runs -> turns (fwd / dQ / dK,dV):
//   d = 128  2 heads, N = 16384   causal 240 -> 211 / 304 -> 280 / 377 -> 246, documents of 700 tokens 64 -> 63 / 76 -> 75 / 79 -> 64
//            3 heads, N = 8192    causal 112 -> 108 / 147 / 158 -> 111;  16 heads, N = 2048 (one round, a unit to a compute unit) as before
//            32 heads on 8 K/V heads, two rows of 2048, shared questions   dK/dV 122 -> 112
//   d = 64   16 heads, N = 2048   causal 28.8 -> 23.5 / 34.7 -> 28.9 / 33.8 -> 28.4, documents 37 -> 31 / 38 -> 37 / 42 -> 40
//            2 heads, N = 16384   causal 165 -> 133 / 194 -> 161 / 218 -> 162;  4 heads, N = 8192, documents 40 -> 41 / 46 -> 47 / 37 -> 36
// Windows of 256 keep their times within 2 to 3 %.  With the blocks of a slice dealt to its XCDs one by one, windows took up to 8 %
// longer (each tile came to every L2) and the three heads' documents 46 instead of 55 us of dK/dV.

// x / n for 0 <= x < 2^31 by a product (Granlund and Montgomery, "Division by Invariant Integers using Multiplication"): the
// divisors are the launch's, and a division takes a workgroup some 30 instructions of its prologue, one behind the other.
struct FmDivisor {
  unsigned n, factor;
  int shift;
};
FM_HOST_DEVICE inline FmDivisor fm_divisor(int n) {
  if (n == 1) return FmDivisor{1, (1u << 31) + 1, 31};
  const int shift = 63 - __builtin_clz(n - 1);   // 31 and the logarithm of n, rounded up
  return FmDivisor{(unsigned)n, (unsigned)((1ull << shift) / (unsigned)n + 1), shift};
}
FM_HOST_DEVICE inline int fm_div(int x, const FmDivisor& d) { return (int)((unsigned long long)(unsigned)x * d.factor >> d.shift); }

enum FmDirectDeal { FM_DEAL_RUNS, FM_DEAL_WHOLE, FM_DEAL_TURNS };
// What a workgroup needs to know is worked out by the host: its way from its number to its unit is a chain of scalar
// instructions in front of everything else.
struct FmDirectOrder {
  FmDirectDeal deal;
  int own, blocks;               // slices of a class, blocks of a slice
  int classes, sharing, chunk;   // m, XCDs of a class, blocks taken together: powers of two, as their logarithms
  int share, odd_units;          // workgroups of an XCD; of them, those that take units one by one: of the slices
  int odd_slice, odd_block;      // from odd_slice on, the blocks from odd_block on
  int turned;                    // (turns) whether a slice begins one XCD further on than the one before
  FmDivisor odd, step, group;    // slices of these units (runs: units of a slice); slices in step otherwise; query heads of a slice
  FmDivisor all;                 // share
};
// at_once: no more units than compute units.
FM_HOST_DEVICE inline FmDirectOrder fm_direct_order(int slices, int group, int blocks, bool at_once) {
  constexpr int kLogXcds = 3, kLogTurns = 2, kLogChunk = 3;
  FmDirectOrder o = {};
  o.own = slices;
  o.blocks = blocks;
  for (o.sharing = kLogXcds; o.classes < kLogXcds && o.own % 2 == 0; o.own /= 2, --o.sharing) ++o.classes;
  const int last = (1 << o.sharing) - 1;
  int odd = o.own, step = o.own;
  o.share = (o.own * group * blocks + last) >> o.sharing;
  if (at_once && o.sharing && o.own > 1) {
    o.deal = FM_DEAL_RUNS;
    odd = group * blocks;
  } else if (o.sharing == 0 || blocks >> (kLogTurns + o.sharing) == 0) {
    o.deal = FM_DEAL_WHOLE;
    odd = o.own & last;
    step = o.own >> o.sharing;
    o.odd_units = o.share - step * group * blocks;
    o.odd_slice = o.own - odd;
  } else {
    o.deal = FM_DEAL_TURNS;
    while (o.chunk < kLogChunk && blocks >> (o.chunk + 1 + kLogTurns + o.sharing)) ++o.chunk;
    const int turns = blocks >> (o.sharing + o.chunk);
    o.turned = turns & 1;
    o.odd_block = turns << (o.sharing + o.chunk);
    o.odd_units = o.share - o.own * group * (turns << o.chunk);
  }
  o.odd = fm_divisor(odd ? odd : 1);
  o.step = fm_divisor(step ? step : 1);
  o.group = fm_divisor(group);
  o.all = fm_divisor(o.share);
  return o;
}
// Workgroups of the launch.
FM_HOST_DEVICE inline int fm_direct_grid(const FmDirectOrder& o) { return 8 * o.share; }
// The slice, member of its group and block that workgroup x takes; block = -1: none.  GROUPED = false: groups of one.
struct FmDirectUnit {
  int slice, member, block;
};
template <bool GROUPED>
FM_HOST_DEVICE inline FmDirectUnit fm_direct_unit(const FmDirectOrder& o, int x) {
  const int xcd = x & 7, p = xcd >> o.classes, at = x >> 3;   // at: which of the XCD's workgroups
  const int first = (xcd & ((1 << o.classes) - 1)) * o.own, group = GROUPED ? (int)o.group.n : 1;
  int slice, i;   // slice of the class; block * group + member
  if (o.deal == FM_DEAL_RUNS) {
    const int unit = p * o.share + at;
    slice = fm_div(unit, o.odd);
    i = slice < o.own ? unit - slice * (int)o.odd.n : group * o.blocks;
  } else {
    // which of the units one by one, or of the others: those come last (turns), or evenly among them (short slices, so that
    // at * odd_units stays below 2^31)
    const bool turns = o.deal == FM_DEAL_TURNS;
    const int odd_before = turns ? at - (o.share - o.odd_units) : fm_div(at * o.odd_units, o.all);
    const bool odd = turns ? odd_before >= 0 : fm_div((at + 1) * o.odd_units, o.all) != odd_before;
    if (odd) {   // a unit to each XCD in turn: every slice's next block, then the block after it
      const int k = (odd_before << o.sharing) + p;
      i = fm_div(k, o.odd);
      slice = o.odd_slice + k - i * (int)o.odd.n;
      i += o.odd_block * group;
    } else if (!turns) {
      i = fm_div(at - odd_before, o.step);
      slice = at - odd_before + (p - i) * (int)o.step.n;
    } else {
      i = fm_div(at, o.step);
      slice = at - i * o.own;
      const int last = (1 << o.sharing) - 1, j = GROUPED ? fm_div(i, o.group) : i;
      const int turn = j >> o.chunk, mine = (p + (o.turned ? slice : 0)) & last;
      const int block = (((turn << o.sharing) + (turn & 1 ? last - mine : mine)) << o.chunk) + (j & ((1 << o.chunk) - 1));
      return FmDirectUnit{first + slice, i - j * group, block};
    }
  }
  const int block = GROUPED ? fm_div(i, o.group) : i;
  return FmDirectUnit{first + slice, i - block * group, block < o.blocks ? block : -1};
}
