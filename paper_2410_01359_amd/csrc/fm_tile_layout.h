// Where a tile's elements lie in LDS, and what the lanes of its copy read.  Plain integer code: the host compiles it too.
#pragma once
#include <cstddef>

#include "fm_interval.h"

#if defined(__HIP__)
#define FM_ALWAYS_INLINE __forceinline__
#else
#define FM_ALWAYS_INLINE inline
#endif

// LDS layout of a [rows][D] bf16 tile, shared by all tile loops.
//
// LDS serves 64 banks x 4 B per clock: 16 lanes of a 128-bit read -- 0-3, 12-15 and 20-27, then 4-11, 16-19 and
// 28-31, then the same of the upper half, as the conflict counter shows -- and 32 lanes of the 64-bit transpose read.
// A tile is groups of 16 rows, a group is panels of 64 bytes of each of its rows (1 KB: what one
// instruction of the direct global->LDS copy writes), and the four 16-byte chunks of a row's part of a panel are
// XORed with 0, 2, 3 or 1, a value to every four rows.  All reads are conflict-free:
//  - operand rows of the 32x32x16 product (32 rows, lanes 0-31 one chunk): 16 lanes have rows of all four values;
//  - operand rows of the 16x16x32 product (16 rows, lanes 16-31 the chunk behind that of lanes 0-15): rows 0-3 and 12-15 of
//    one chunk meet rows 4-11 of its neighbour (chunk ^ 1), four different slots because 0, 1 and 2 ^ 1, 3 ^ 1 differ.  With 0, 2, 1, 3
//    they met in pairs, 4 clocks a read, 40 % of the dQ loop's LDS cycles at d = 128;
//  - transpose reads: 4 rows x 64 bytes of a panel are one bank line, 8 rows x 32 bytes two halves of different bit 1.
// dQ, prefix 4096 of 32768, 16 heads, d = 128: LDS cycles 1378e6 -> 831e6, of them conflicts 548e6 -> 1.6e6 (the results'
// staging), time unchanged (5074 -> 5076 us: power); d = 64, 1024 units of 1024 to 16384 tokens, 0.4 to 1.5 % faster.
// off(row + 16*m, col) == off(row, col) + 16*m*RS, and a panel further on is 1 KB further on, so callers precompute
// the lane-dependent part once and nearly all of a tile's reads differ from it by an instruction's immediate offset.
template <int D>
struct TileLayout {
  static constexpr int RS = D * 2;       // bytes per row
  static constexpr int PANELS = D / 32;  // of 64 bytes per row
  static FM_HOST_DEVICE FM_ALWAYS_INLINE int swz(int row) { return ((row >> 1 ^ row >> 2) & 2) | ((row >> 3) & 1); }
  static FM_HOST_DEVICE FM_ALWAYS_INLINE int off(int row, int byte_col) {
    return (row >> 4) * (16 * RS) + (byte_col >> 6) * 1024 + (row & 15) * 64 +
           (((((byte_col >> 4) & 3) ^ swz(row)) << 4) | (byte_col & 15));
  }
  // off(row, col0 + colc) from off(row, col0), for a constant colc that is a multiple of 32 and col0 < 32 (operand
  // rows) or a multiple of 64 and col0 < 64 (transpose reads).
  static FM_HOST_DEVICE FM_ALWAYS_INLINE unsigned add_col(unsigned base, unsigned colc) {
    return (base ^ (colc & 32)) + (colc >> 6) * 1024;
  }
};

// Asynchronous global->LDS copy of a [64][D] bf16 tile (global row stride D)
// into TileLayout<D> order by a 4-wave workgroup.  Wave w copies rows
// 16w..16w+15, a contiguous block on both sides, with NINST instructions of
// 64 x 16 B = 1 KB each straight into LDS (no staging registers), a panel of 16 rows each; the order of rows and
// chunks is applied on the global-address side.  The LDS destination of such an
// instruction is M0 + immediate offset + 16 * lane and the same immediate is
// added to the global address, so one M0 value (async_window) serves all of a
// wave's instructions for a tile: rewriting M0 costs the issuing wave about as
// much as the copy itself.  CopyLanes holds the per-lane source byte offset
// of each instruction (relative to the wave's row block); the swizzle repeats
// every 16 rows, so it does not depend on the wave.
template <int D>
struct CopyLanes {
  using L = TileLayout<D>;
  static constexpr int NINST = L::PANELS;     // instructions per wave and tile
  // Instruction s carries the immediate s * 1024 on both sides, where its panel is 64 s bytes further on in global memory:
  // the difference goes into the lane offset, and what keeps that from turning negative into the base (wave_base).
  static constexpr int BIAS = (NINST - 1) * (1024 - 64);
  unsigned v[NINST];
  // grs: bytes between consecutive rows of the global tensor (TileLayout::RS when it is contiguous).
  FM_HOST_DEVICE FM_ALWAYS_INLINE void init(int lane, int grs = L::RS) {
#pragma unroll
    for (int s = 0; s < NINST; ++s) v[s] = lane / 4 * grs + source_col(lane, s) - s * 1024 + BIAS;
  }
  // Byte column of a row that a lane of instruction s copies (row lane / 4 of the wave's 16).
  static FM_HOST_DEVICE FM_ALWAYS_INLINE int source_col(int lane, int s) { return s * 64 + ((lane % 4 ^ L::swz(lane / 4)) << 4); }
  // What the lane offsets count from: row 0 of a tensor's slice -> this wave's row 0 of the tile at row 0.
  static FM_HOST_DEVICE FM_ALWAYS_INLINE const char* wave_base(const void* slice, int wave, int grs) {
    return (const char*)slice + (size_t)(wave * 16) * grs - BIAS;
  }
};
