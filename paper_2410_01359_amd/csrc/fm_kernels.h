// Host-side launchers of the gfx950 FlashMask kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <initializer_list>

#include "fm_direct_order.h"

// The tile loops draw their work units from FM_QUEUES interleaved queues (one per XCD).
constexpr int FM_QUEUES = 8;
// Number of queue slots for `units` work units.
// Slices (batch row, head) of a queue that are ranked together, longest first; a queue works its
// groups off one after the other.
constexpr int FM_QUEUE_CHUNK = 2;
// Slots of a pass's queues: FM_QUEUES x the longest queue.  Slices that do not fill a round of
// 8 queues are shared between 2, 4 or 8 queues block by block, which can make a queue up to 3 units
// longer than an eighth of all units.
inline int fm_order_slots(int units) { return ((units + FM_QUEUES - 1) / FM_QUEUES + 3) * FM_QUEUES; }
// Bytes of a pass's queue area: one 16-byte record per slot, then the FM_QUEUES queue counters.
inline size_t fm_order_bytes(int units) { return (size_t)fm_order_slots(units) * 16 + FM_QUEUES * 4; }
// Raise the dynamic LDS limits of a tile loop's kernels of one shape class (head dimension, ragged or not, general
// layout or not) once per device (the attribute belongs to the device's copy of the kernel).  All cuts of the work
// together: one call prepares its class for a graph capture, whichever cut the captured sizes take.  `done` is the
// class's own flag array, one flag per device.
constexpr int FM_MAX_DEVICES = 64;
struct FmLdsLimit {
  const void* kernel;
  int bytes;
};
inline hipError_t fm_allow_lds(std::initializer_list<FmLdsLimit> limits, bool (&done)[FM_MAX_DEVICES]) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  // The flags are shared by every host thread that calls the library: atomic accesses; two threads
  // that both find a flag clear both set the attributes, which is harmless (same values).
  if (dev >= 0 && dev < FM_MAX_DEVICES && __atomic_load_n(&done[dev], __ATOMIC_ACQUIRE)) return hipSuccess;
  for (const FmLdsLimit& l : limits) {
    e = hipFuncSetAttribute(l.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, l.bytes);
    if (e != hipSuccess) return e;
  }
  if (dev >= 0 && dev < FM_MAX_DEVICES) __atomic_store_n(&done[dev], true, __ATOMIC_RELEASE);
  return e;
}
// Compute units of the current device (looked up once per device), 0 on failure.
inline int fm_compute_units() {
  static int cached[FM_MAX_DEVICES] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= FM_MAX_DEVICES) return 0;
  int n = __atomic_load_n(&cached[dev], __ATOMIC_RELAXED);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    __atomic_store_n(&cached[dev], n, __ATOMIC_RELAXED);
  }
  return n;
}
// A pass's unit queues as its tile loop sees them.
struct FmQueue {
  int* order;    // slot records {unit, first live block, one past the last, 0}, unit = -1: none; then the counters
  int slots;     // records (fm_order_slots)
  int tickets;   // records that can hold a unit: FM_QUEUES x the longest queue
  int first;     // tickets that are the number of the workgroup that takes them: those of the workgroups that run
                 // from the start.  The order in which the others start decides theirs.
};
// Queues of `slices` slices (batch row, K/V head) of `units` units each.  How the slices that do not fill a round
// of 8 queues are shared (fm_queue_of): queue 0 has a half, a quarter and an eighth of them, rounded up.
inline FmQueue fm_queue(int* order, int slices, int units) {
  const int r = slices % FM_QUEUES;
  const int longest = slices / FM_QUEUES * units + ((r & 4) ? (units + 1) / 2 : 0) + ((r & 2) ? (units + 3) / 4 : 0) +
                      ((r & 1) ? (units + 7) / 8 : 0);
  return FmQueue{order, fm_order_slots(slices * units), longest * FM_QUEUES, 0};
}
// The queues for a launch that runs `per_cu` workgroups on each compute unit.
inline FmQueue fm_queue_for_launch(FmQueue q, int per_cu) {
  const int g = fm_compute_units() * per_cu / FM_QUEUES * FM_QUEUES;
  q.first = g < q.tickets ? g : q.tickets;
  return q;
}
// Workgroups of a tile-loop launch: one per ticket, and where not all of them run from the start a reserve of one
// eighth, through which the XCDs that finish their own queue early take units from the others (a workgroup that
// finds every queue empty ends at once).
inline int fm_launch_grid(const FmQueue& q) { return q.first == q.tickets ? q.tickets : q.tickets + fm_order_slots(q.tickets / 8); }
// Workgroups of a persistent launch (every workgroup works units off until the queues are empty): those that run
// from the start (one per ticket if the number of compute units is not known).
inline int fm_persistent_grid(const FmQueue& q) { return q.first > 0 ? q.first : q.tickets; }
// How a tile loop's work is cut into workgroups.
enum FmUnits {
  FM_QUEUED,          // units of 128 rows (keys) off the unit queues, which the setup launches build
  FM_DIRECT,          // the same units without setup launches (see fm_common.h)
  FM_DIRECT_HALVED,   // units of 64 rows (keys), their tiles shared by two pairs of waves
  FM_DIRECT_PAIRED,   // units of 128 rows, their tiles shared by two groups of four waves (row-parallel loops, d = 128)
};
constexpr int fm_groups(FmUnits u) { return u == FM_DIRECT_HALVED || u == FM_DIRECT_PAIRED ? 2 : 1; }
constexpr int fm_group_waves(FmUnits u) { return u == FM_DIRECT_HALVED ? 2 : 4; }
// Workgroups of 128-row (128-key) units on a compute unit, four waves each.
constexpr int fm_fwd_per_cu(int d) { return d == 64 ? 3 : 2; }
constexpr int FM_DQ_PER_CU = 2;
constexpr int fm_dkdv_per_cu(int d) { return d == 64 ? 2 : 1; }
// The lines between the cuts.  The host does not know the mask, so they are drawn by the geometric mean of times over six:
// causal, a prefix of an eighth, causal documents of 700 tokens, eight documents both ways (two below 2048 tokens), a window of
// 256, shared questions.  A ratio is that mean, of a cut over the queues unless it says otherwise, each with its setup; a pair is
// forward / backward with the other loops' cuts as they are, or (in all loops) with all of them cut that way.
// Several lines lie short of where the ratios cross: they were drawn before the blocks of all slices went in step, and the
// sizes beyond are what the tests name to reach the queues.  What direct units measure there stands beside each.
//
// Sequences so short that what a unit does hardly differs gain nothing from an order, and the setup launch is a good part of
// their time.  In all loops: d = 128, 1024 units, N = 512 0.77 / 0.90, N = 128 0.64 / 0.80;   d = 64, 2048 units, N = 512 0.67 / 0.72,
// N = 128 0.50 / 0.59.  Beyond: d = 128, 2048 units, N = 512 0.78 / 0.93;   d = 64, 4096 units, N = 512 0.68 / 0.73.
inline bool fm_short_direct(long long units, int d, int N, long long cus) {
  return N <= 512 && units <= (d == 64 ? 8 : 4) * cus;
}
// Where the blocks of all slices go in step (fm_direct_order.h), up to three units a compute unit need no order at short and
// medium lengths either, rows and keys alike (`units` counts row blocks, so that the backward's loops cross the line together and
// no setup launch is left for one of them).  In all loops:
//   d = 128  576 units, N = 1000  0.68 / 0.76;   640, N = 1024  0.73 / 0.80, N = 2048  0.78 / 0.82;   768, N = 1500  0.79 / 0.82, N = 2000  0.87 / 0.89;
//            odd counts of slices: 150 of 600 tokens 0.70 / 0.80, 75 of 1024 0.63 / 0.75, 51 of 1900 0.83 / 0.81, 45 of 2048 0.77 / 0.80
//   d = 64   150 slices of 600 tokens 0.70 / 0.73, 75 of 1024 0.61 / 0.67, 17 of 4096 0.75 / 0.85, 24 of 4096 0.76 / 0.83, 32 of 3000 0.90 / 0.90
//   grouped heads, 40 on 10, N = 2048  d = 128 0.78 / 0.93, d = 64 0.71 / 0.90;   three rows of 42 on 14  0.92 / 0.92, 0.79 / 0.92
// Single masks: documents both ways take up to 1.12 times as long (backward, three rows of 14 K/V heads, 23 heads of 4096 at d = 64).
// Beyond, rows alone: d = 128, N = 4096, 512 units 0.91 / 0.95, 768 0.85 / 0.97;  N = 8192, 512 units 0.94 / 0.97;  two rows of 32 on 8
// heads, N = 4096 0.97 / 1.00.  In all loops, 1024 units: d = 128, N = 1024 0.75 / 0.90, N = 2048 0.85 / 0.90;  d = 64 0.67 / 0.74, 0.73 / 0.80.
inline bool fm_in_step(long long units, int d, int N, long long cus) { return units <= 3 * cus && N <= (d == 128 ? 2048 : 4096); }
// The cut of a row-parallel loop over `units` units of 128 rows in groups of `group` query heads to a K/V head, `per_cu` of
// which one of `cus` compute units holds, at sequence length n.  What is weighed: the setup launch (4 us up to N = 4096, 8 us
// beyond), the longest chain of tiles (halved by two groups), waves per SIMD, and building the list from the bound vectors instead
// of the table (which grows with N; ragged lengths load the bounds 4 bytes at a time).  Halved, paired, direct (rows alone):
//   d = 128  128 units, N = 2048   0.60 / 0.74, 0.72 / 0.85, 0.81 / 0.91;   N = 16384  0.69 / 0.78, 0.79 / 0.87, 0.99 / 1.00
//            144 units, N = 2048   0.73 / 0.86, 0.72 / 0.86, 0.81 / 0.91
//            256 units, N = 512    0.78 / 0.91, 0.69 / 0.86, 0.67 / 0.83;   N = 2048   0.83 / 0.92, 0.74 / 0.88, 0.82 / 0.92
//                       N = 8192   0.85 / 0.91, 0.76 / 0.88, 0.91 / 0.96;   N = 32768  1.01 / 1.05, 0.85 / 0.97, 1.08 / 1.09
//                       N = 16307  1.06 / 1.01, 0.89 / 0.93, 1.03 / 1.02;   N = 32691  1.20 / 1.09, 0.96 / 0.98, 1.14 / 1.08
//            320 units, N = 2048          -   0.68 / 0.84, 0.69 / 0.84;   512 units, N = 1024   -   0.88 / 0.96, 0.71 / 0.87
//   d = 64, halved, direct
//            256 units, N = 2048   0.62 / 0.77, 0.81 / 0.88;   N = 8192   0.66 / 0.79, 0.92 / 0.95;   N = 32768  0.81 / 0.90, 1.12 / 1.09
//                       N = 16307  0.94 / 0.97, 1.06 / 1.05;   N = 32691  1.09 / 1.11, 1.18 / 1.15
//            512 units, N = 512    0.73 / 0.86, 0.60 / 0.75;   N = 1024   0.72 / 0.84, 0.66 / 0.80;   N = 2048   0.74 / 0.87, 0.71 / 0.85
//            (320:                                                                                               0.60 / 0.75, 0.68 / 0.81)
//                       N = 4096   0.90 / 0.93, 0.91 / 0.92;   N = 8192   0.94 / 0.94, 0.94 / 0.95;   N = 16384  1.03 / 0.99, 1.02 / 0.99
//                       N = 8115   1.20 / 1.08, 1.05 / 1.01;   N = 16307  1.36 / 1.18, 1.19 / 1.10
// Windows lose most (forward, 32691 tokens: paired at d = 128 42 us for 27, halved at d = 64 64 for 22).  The lines carry no raggedness: at d = 64 ragged
// lengths of 8115 tokens (512 units) and 32691 (256 units) are halved where the queues are faster.
// Forward units at d = 64 that all run at once, three to a compute unit, direct over queued: full blocks up to 8192, 513 to 768 units,
// 0.79 to 0.96, grouped heads 0.92 to 1.00;  ragged up to 5120 0.83 to 1.03 (five sizes, mean 0.93), beyond 0.89 to 1.07 (ten, 0.99;
// windows 1.15 to 1.4);  ragged with grouped heads up to 5120 0.95 to 1.03 (six, 0.99), beyond 1.00 to 1.10 (nine, 1.05): queued.
inline FmUnits fm_row_units(long long units, int group, int per_cu, int d, int n, long long cus) {
  const int N = (n + 127) / 128 * 128;
  if (d == 128) {
    if (2 * units <= cus) return FM_DIRECT_HALVED;
    if (units <= cus) return FM_DIRECT_PAIRED;
    return fm_in_step(units, d, N, cus) || fm_short_direct(units, d, N, cus) ? FM_DIRECT : FM_QUEUED;
  }
  if (units <= cus) return FM_DIRECT_HALVED;
  if (units <= 2 * cus && N > 1024) return N <= 8192 ? FM_DIRECT_HALVED : FM_QUEUED;
  const int at_once_to = n != N && group > 1 ? 5120 : 8192;
  return fm_in_step(units, d, N, cus) || (units <= per_cu * cus && N <= at_once_to) || fm_short_direct(units, d, N, cus) ? FM_DIRECT : FM_QUEUED;
}
// The same for the dK/dV loop over units of 128 keys of `group` query heads each (a chain `group` times as long; lists
// are built from the unit's own keys' bounds at any N).  Backward, keys alone, halved, direct; of 1, 2, 4 and 8 query heads:
//   d = 128  128 units, N = 2048   0.75, 0.89   -   0.73, 0.96   -;                  N = 16384  0.75, 0.93
//            256 units, N = 512    0.92, 0.84   0.96, 0.88   0.96, 0.94   1.00, 1.00;   N = 1024   0.91, 0.87   0.91, 0.91   0.96, 1.00   0.95, 1.00
//                       N = 2048   0.90, 0.90   0.90, 0.94   0.93, 1.00   0.92, 1.00;   N = 8192   0.87, 0.92   0.90, 1.00   0.86, 0.99   0.86, 0.99
//                       N = 16384  0.87, 0.93   0.88, 0.99   0.86, 0.99   0.86, 0.99;   N = 24576  0.83, 0.95   0.84, 1.00   0.79, 1.00   0.78, 1.00
//                       N = 24500  0.84, 0.96   0.84, 1.00   0.80, 1.00   0.80, 1.00;   N = 32768  0.87, 0.95;   N = 32691  0.89, 0.96
//            512 units, N = 1024   0.94, 0.81;   N = 2048   0.88, 0.81;   N = 4096   0.99, 0.94
//                       N = 8192   0.96, 0.93   0.94, 0.94   0.93, 0.94   0.93, 0.95;   N = 16384  0.95, 0.94   0.93, 0.94   0.91, 0.94   0.90, 0.94
//                       N = 16290  0.96, 0.93   0.96, 0.93   0.94, 0.93   0.92, 0.92;   N = 32768  0.94, 0.94
//            384 units, N = 16384  0.97, 0.98   0.94, 0.98   0.91, 0.97   0.90, 0.97;   400 units, N = 10240  0.97, 0.94   0.96, 0.95   0.94, 0.95   0.92, 0.93
//   d = 64   256 units, N = 2048   0.78, 0.86
//            512 units, N = 1024   0.84, 0.80   -   0.91, 0.92;   N = 2048   0.83, 0.83   -   0.87, 0.91;   N = 4096   0.91, 0.92
//                       N = 8192   0.89, 0.94   -   0.92, 1.00;   N = 16384  0.94, 1.00   -   0.89, 1.00;   N = 32768  0.92, 0.99
//                       N = 16307  0.94, 1.01;   N = 32691  0.92, 0.99   -   0.88, 1.00;   480 units, N = 20480  0.96, 1.02   -   0.92, 1.03
// Halved units of a full round copy each row tile twice as often and run in two rounds: that pays while the longest chain
// decides.  Beyond 16384 tokens full rounds are queued all the same (ragged ones at d = 128 halved).  Two rounds of keys up to 16384
// tokens, single masks: causal 0.82 to 0.93, windows 0.87 to 0.99; eight documents both ways, ten draws, 0.94 to 1.12, one of
// them at 3 K/V heads of 16384 tokens 1.25 (8 query heads 1.40).
inline FmUnits fm_key_units(long long units, int group, int d, int N, long long cus) {
  const long long slots = fm_dkdv_per_cu(d) * cus;
  const int padded = (N + 127) / 128 * 128;
  const bool ragged = N != padded;
  if (2 * units <= slots) return FM_DIRECT_HALVED;
  if (units <= slots) {
    if ((long long)padded * group <= (d == 128 ? 2048 : 1024)) return FM_DIRECT;
    return (ragged && d == 128) || N <= 16384 ? FM_DIRECT_HALVED : FM_QUEUED;
  }
  return (d == 128 && units <= 2 * slots && N <= 16384) || fm_in_step(units * group, d, padded, cus) ||
                 fm_short_direct(units, d, padded, cus)
             ? FM_DIRECT
             : FM_QUEUED;
}
// Tile shapes (rows x key columns) each pass classifies at.
constexpr int FM_FWD_BR = 128, FM_FWD_BC = 64;
constexpr int FM_DQ_BR = 128;
// Key columns per tile of the dQ pass: at d = 64 a 128-key tile has the bytes (and the MFMAs) of a 64-key tile at
// d = 128, so that a tile's fixed work (copies' set-up, list entry, wait, barrier) is spread over as much math.
constexpr int fm_dq_bc(int d) { return d == 64 ? 128 : 64; }
constexpr int FM_DKDV_BR = 64, FM_DKDV_BC = 128;

// What the columns past the end of a sequence whose length is no multiple of 128 count as in a pass's table.
enum FmPads {
  FM_PADS_NONE,     // nothing: a block covers the columns that exist (dK/dV units, whose lanes past the last key copy it)
  FM_PADS_MASKED,   // masked for every row by both pairs (the row-parallel loops, see pad_column)
};
// One pass's setup buffers (in the workspace) and tile shape.
struct FmSetup {
  int block_r, block_c;
  int* minmax;   // int[B][8][T_c]
  int* work;     // int[B * T], T = row blocks resp. key blocks
  int* range;    // int[2 * B * T]: first live block and one past the last live block of every unit (0, 0 if none)
  int* order;    // fm_order_bytes(B * H * T) bytes: slot records {unit, first, last, 0}, then the counters (zeroed here)
  FmPads pads;
};
// Workgroups of the queue-building launch: per queue, one for every FM_QUEUE_CHUNK whole slices and one
// for its part of the slices left over, its unused slots and its counter.
inline int fm_order_grid(int B, int H) {
  return FM_QUEUES * (((B * H) / FM_QUEUES + FM_QUEUE_CHUNK - 1) / FM_QUEUE_CHUNK + 1);
}

// Launches of the setup of one pass, or of the backward's two together, with B rows of H slices (K/V heads) at the padded
// length Np: one launch (setup_kernel) or three (tables, work, queues).  One launch repeats the table in every workgroup.
// Training step, three -> one in each direction, d = 64 / 128: N = 512 68 -> 58 / 78 -> 70 us, N = 2048 118 -> 109 /
// 153 -> 146 us, N = 4096 no difference within 3 us; with more passes over the columns (the work grows with N^2 as well)
// it lost 4 us at N = 8192 and 10 to 15 us at N = 16384.  With more workgroups of 1024 threads than compute units the
// repetition costs more than the launches: forward / backward, one | three launches, d = 128: 200 | 400 workgroups,
// N = 512 74 / 203 | 77 / 201 us, N = 1024 178 / 471 | 180 / 467; 264 | 528, N = 256 46 / 120 | 46 / 118; 1032 | 2064,
// N = 128 89 / 239 | 79 / 219, N = 512 349 / 935 | 340 / 916; 72 | 144, N = 1024 74 / 182 | 76 / 185.
constexpr int FM_ONE_LAUNCH_LENGTH = 4096;
inline int fm_setup_launches(int passes, int B, int H, int Np, int cus) {
  return Np <= FM_ONE_LAUNCH_LENGTH && passes * fm_order_grid(B, H) <= cus ? 1 : 3;
}
// A pass's whole setup: table, work and live range of every unit, unit queues.  cols: the units are key blocks (they
// count K/V heads), else row blocks.  One launch writes minmax and order only.
hipError_t fm_launch_setup(const int* lts, const int* lte, const int* uts, const int* ute, int B, int H, int Hk, int N,
                           int Np, const FmSetup& pass, bool cols, hipStream_t stream);
// The same for the dQ pass `rows` and the dK/dV pass `cols` together.
hipError_t fm_launch_bwd_setup(const int* lts, const int* lte, const int* uts, const int* ute, int B, int H, int Hk,
                               int N, int Np, const FmSetup& rows, const FmSetup& cols, hipStream_t stream);
// Tables of ceil(Np / block_c) key blocks per batch row; the columns [N, Np), and a ragged last block's beyond N, count
// as `pads` says.
hipError_t fm_launch_preprocess(const int* lts, const int* lte, const int* uts, const int* ute, int B, int N, int Np,
                                int block_c, FmPads pads, int* minmax, hipStream_t stream);
hipError_t fm_launch_classify(const int* minmax, int B, int N, int block_r, int block_c, uint8_t* cls,
                              hipStream_t stream);


// Measurement aid (fm_probe.hip): `workgroups` x 4 waves each issue iters x fm_mfma_ceiling_ops_per_iter()
// MFMA slots (shape 0: one 32x32x16 bf16 instruction; 1: two of the 16x16x32 shape, the same floating-point
// operations; 2: shape 0 plus the forward loop's side work per MFMA) on the operands given
// (2 * 8 * 64 * 16 bytes), one float per thread into sink.
hipError_t fm_launch_mfma_ceiling(const void* operands, float* sink, int workgroups, int iters, int shape,
                                  hipStream_t stream);
int fm_mfma_ceiling_ops_per_iter();
// Measurement aid: `workgroups` workgroups each add `tiles` 64 x 128 fp32 tiles into acc
// ([heads][n_tiles][64][128] floats) with no-return atomic adds.
hipError_t fm_launch_atomic_ceiling(float* acc, int n_tiles, int tiles, int heads, int workgroups, hipStream_t stream);

// Element strides of a bf16 tensor indexed [batch][head][row][d] (d contiguous).
struct FmStride {
  long long b, h, n;
};

// `general` selects the kernel instantiations that honour the stride fields and Hk (number of
// K/V heads, H % Hk == 0: query head h reads K/V head h / (H / Hk)); otherwise every tensor is
// contiguous [B,H,N,d], Hk == H, and the strides are compile-time constants of the kernels.
// N is the true sequence length (stride of the tensors and of the bound vectors), Np = N rounded up to a
// multiple of 128: the length the tile loops and the tables work at.  When Np > N the extra key columns count as
// FmPads says (rows' loops: masked for every row); rows are classified up to N only.
// The strides (96 bytes forward, 192 backward) travel to the GEN kernels only: each launch copies its arguments, and the host's
// work is what a small call takes.  Training step, 2 heads of 512 tokens, d = 64, three launches: 0.3 of 27.4 us.
template <bool GEN>
struct FmFwdStrides {
  FmStride sq, sk, sv, so;
};
template <>
struct FmFwdStrides<false> {
  static constexpr FmStride sq{}, sk{}, sv{}, so{};   // never read
};
struct FmFwdCommon {
  const void *q, *k, *v;
  const int *lts, *lte, *uts, *ute;   // [B][N]
  const int* minmax;  // [B][8][T_c] at FM_FWD_BC
  FmQueue queue;      // units (b*H + h)*T_r + i; a row block is fully masked outside its key blocks [first, last)
  void* out;
  float* lse;
  float scale;
  int B, H, N, Np, d;
  FmUnits units;      // direct ones: minmax and queue are not used, but
  FmDirectOrder order;   // (filled in by the launch)
  bool general;
  int Hk;
};
template <bool GEN>
struct FmFwdKernelArgs : FmFwdCommon, FmFwdStrides<GEN> {};
using FmFwdArgs = FmFwdKernelArgs<true>;
hipError_t fm_launch_fwd(const FmFwdArgs& a, hipStream_t stream);

template <bool GEN>
struct FmBwdStrides {
  FmStride sq, sk, sv, so, sdo, sdq, sdk, sdv;
};
template <>
struct FmBwdStrides<false> {
  static constexpr FmStride sq{}, sk{}, sv{}, so{}, sdo{}, sdq{}, sdk{}, sdv{};
};
struct FmBwdCommon {
  const void *q, *k, *v, *out, *dout;
  const float* lse;
  const int *lts, *lte, *uts, *ute;
  const int* minmax_dq;    // [B][8][T_c] at fm_dq_bc(d)
  FmQueue queue_dq;        // of the dQ pass (live key-block range per row block)
  const int* minmax_dkdv;  // [B][8][T_c] at FM_DKDV_BC
  FmQueue queue_dkdv;      // of the dK/dV pass (live row-block range per key block)
  float* dvec;             // -D = -rowsum(dO o O), [B,H,Np] (stored negated; 0 in the padding): written by the
                           // dQ loop's prologue, read by the dK/dV loop
  float* lse2;             // lse * log2(e), +inf where lse = -inf and in the padding, [B,H,Np]: likewise
  void *dq, *dk, *dv;
  float scale;
  int B, H, N, Np, d;
  FmUnits units_dq, units_dkdv;   // direct ones: the pass's minmax and queue are not used, but
  FmDirectOrder order;            // of the pass that is launched (filled in by the launch)
  bool general;
  int Hk;
};
template <bool GEN>
struct FmBwdKernelArgs : FmBwdCommon, FmBwdStrides<GEN> {};
using FmBwdArgs = FmBwdKernelArgs<true>;
// What a kernel gets of a call's arguments.
template <bool GEN>
inline FmFwdKernelArgs<GEN> fm_kernel_args(const FmFwdArgs& a) {
  if constexpr (GEN) return a;
  else return {a, {}};
}
template <bool GEN>
inline FmBwdKernelArgs<GEN> fm_kernel_args(const FmBwdArgs& a) {
  if constexpr (GEN) return a;
  else return {a, {}};
}
hipError_t fm_launch_bwd_dq(const FmBwdArgs& a, hipStream_t stream);
hipError_t fm_launch_bwd_dkdv(const FmBwdArgs& a, hipStream_t stream);
