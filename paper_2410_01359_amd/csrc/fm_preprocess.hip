// Preprocessing (Section 4.2): per key-block min/max of the four bound vectors,
// the exported tile-class dump (Equation 4), the per-unit work counts, and
// the unit queues built from them.
#include <climits>

#include "fm_common.h"
#include "fm_kernels.h"

namespace fm {

// One wave per (batch row, key block).  Lanes stride over the block's columns,
// then a butterfly over the 64 lanes leaves the 8 results in every lane.
__device__ __forceinline__ void preprocess_body(const int* __restrict__ lts, const int* __restrict__ lte,
                                                const int* __restrict__ uts, const int* __restrict__ ute, int n,
                                                FmPads pads, int block_c, int t_c, int total_blocks,
                                                int* __restrict__ minmax, int block) {
  const int lane = threadIdx.x & 63;
  const int blk = block * 4 + (threadIdx.x >> 6);
  if (blk >= total_blocks) return;
  const int b = blk / t_c, j = blk - b * t_c;
  const int c0 = j * block_c;
  const int c1 = min(c0 + block_c, n);
  const int* vec[4] = {lts + (size_t)b * n, lte + (size_t)b * n, uts + (size_t)b * n, ute + (size_t)b * n};
  int mx[4], mn[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    mx[a] = INT32_MIN;
    mn[a] = INT32_MAX;
  }
  if (pads != FM_PADS_NONE && c0 + block_c > n) {   // the block's columns past the end of the sequence
#pragma unroll
    for (int a = 0; a < 4; ++a) mx[a] = mn[a] = pad_value(pads, a, 0);
  }
  for (int c = c0 + lane; c < c1; c += 64) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int x = vec[a][c];
      mx[a] = max(mx[a], x);
      mn[a] = min(mn[a], x);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      mx[a] = max(mx[a], __shfl_xor(mx[a], off, 64));
      mn[a] = min(mn[a], __shfl_xor(mn[a], off, 64));
    }
  }
  if (lane == 0) {
    int* out = minmax + (size_t)b * 8 * t_c;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      out[(2 * a) * t_c + j] = mx[a];
      out[(2 * a + 1) * t_c + j] = mn[a];
    }
  }
}

__global__ __launch_bounds__(256) void preprocess_kernel(const int* __restrict__ lts, const int* __restrict__ lte,
                                                         const int* __restrict__ uts, const int* __restrict__ ute,
                                                         int n, FmPads pads, int block_c, int t_c, int total_blocks,
                                                         int* __restrict__ minmax) {
  preprocess_body(lts, lte, uts, ute, n, pads, block_c, t_c, total_blocks, minmax, blockIdx.x);
}

// The tables of two block widths in one launch (the backward's two loops tile the keys differently):
// workgroups [0, blocks_a) build table a, the rest table b.
__global__ __launch_bounds__(256) void preprocess2_kernel(const int* __restrict__ lts, const int* __restrict__ lte,
                                                          const int* __restrict__ uts, const int* __restrict__ ute,
                                                          int n, int np, int batch, int block_c_a, FmPads pads_a,
                                                          int* __restrict__ minmax_a, int blocks_a, int block_c_b,
                                                          FmPads pads_b, int* __restrict__ minmax_b) {
  const bool first = (int)blockIdx.x < blocks_a;
  const int block_c = first ? block_c_a : block_c_b;
  const int t_c = (np + block_c - 1) / block_c;
  preprocess_body(lts, lte, uts, ute, n, first ? pads_a : pads_b, block_c, t_c, batch * t_c, first ? minmax_a : minmax_b,
                  first ? blockIdx.x : blockIdx.x - blocks_a);
}

__global__ __launch_bounds__(256) void classify_kernel(const int* __restrict__ minmax, int n, int block_r, int t_r,
                                                       int t_c, uint8_t* __restrict__ cls) {
  const int b = blockIdx.z, i = blockIdx.y;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= t_c) return;
  const MinMax8 t = load_minmax(minmax + (size_t)b * 8 * t_c, t_c, j);
  const int r0 = i * block_r;
  const int r1 = min(r0 + block_r, n);
  cls[((size_t)b * t_r + i) * t_c + j] = (uint8_t)classify_tile(r0, r1, t);
}

// Work of one row block = number of key blocks that are not fully masked, and
// the range of key blocks that contains them (the tile loops only scan that).
// One wave per (batch row, row block); lanes stride over the key blocks.
__device__ __forceinline__ void row_work_body(const int* __restrict__ minmax, int n, int block_r, int t_r, int t_c,
                                              int total_units, int* __restrict__ work, int* __restrict__ range,
                                              int block) {
  const int lane = threadIdx.x & 63;
  const int u = block * 4 + (threadIdx.x >> 6);
  if (u >= total_units) return;
  const int b = u / t_r, i = u - b * t_r;
  const int r0 = i * block_r, r1 = min(r0 + block_r, n);
  const int* table = minmax + (size_t)b * 8 * t_c;
  int cnt = 0, lo = t_c, hi = 0;
#pragma unroll 8   // the table loads of several iterations in flight: the scan is bound by their latency
  for (int j = lane; j < t_c; j += 64)
    if (classify_tile(r0, r1, load_minmax(table, t_c, j)) != T_FULLY) {
      ++cnt;
      lo = min(lo, j);
      hi = j + 1;
    }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    cnt += __shfl_xor(cnt, off, 64);
    lo = min(lo, __shfl_xor(lo, off, 64));
    hi = max(hi, __shfl_xor(hi, off, 64));
  }
  if (lane == 0) {
    work[u] = cnt;
    range[2 * u] = cnt ? lo : 0;
    range[2 * u + 1] = hi;
  }
}

__global__ __launch_bounds__(256) void row_work_kernel(const int* __restrict__ minmax, int n, int block_r, int t_r,
                                                       int t_c, int total_units, int* __restrict__ work,
                                                       int* __restrict__ range) {
  row_work_body(minmax, n, block_r, t_r, t_c, total_units, work, range, blockIdx.x);
}

// Work of one key block = number of row blocks that are not fully masked.
__device__ __forceinline__ void col_work_body(const int* __restrict__ minmax, int n, int block_r, int t_r, int t_c,
                                              int total_units, int* __restrict__ work, int* __restrict__ range,
                                              int block) {
  const int lane = threadIdx.x & 63;
  const int u = block * 4 + (threadIdx.x >> 6);
  if (u >= total_units) return;
  const int b = u / t_c, j = u - b * t_c;
  const MinMax8 t = load_minmax(minmax + (size_t)b * 8 * t_c, t_c, j);
  int cnt = 0, lo = t_r, hi = 0;
  for (int i = lane; i < t_r; i += 64) {
    const int r0 = i * block_r, r1 = min(r0 + block_r, n);
    if (classify_tile(r0, r1, t) != T_FULLY) {
      ++cnt;
      lo = min(lo, i);
      hi = i + 1;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    cnt += __shfl_xor(cnt, off, 64);
    lo = min(lo, __shfl_xor(lo, off, 64));
    hi = max(hi, __shfl_xor(hi, off, 64));
  }
  if (lane == 0) {
    work[u] = cnt;
    range[2 * u] = cnt ? lo : 0;
    range[2 * u + 1] = hi;
  }
}

__global__ __launch_bounds__(256) void col_work_kernel(const int* __restrict__ minmax, int n, int block_r, int t_r,
                                                       int t_c, int total_units, int* __restrict__ work,
                                                       int* __restrict__ range) {
  col_work_body(minmax, n, block_r, t_r, t_c, total_units, work, range, blockIdx.x);
}

// One pass's work pre-pass as arguments, so that the backward can run both of its passes' in one launch.
struct WorkJob {
  const int* minmax;
  int block_r, t_r, t_c, total_units;
  int* work;
  int* range;
};
// workgroups [0, blocks_rows) count per row block (job `rows`), the rest per key block (job `cols`)
__global__ __launch_bounds__(256) void work2_kernel(WorkJob rows, int blocks_rows, WorkJob cols, int n) {
  if ((int)blockIdx.x < blocks_rows)
    row_work_body(rows.minmax, n, rows.block_r, rows.t_r, rows.t_c, rows.total_units, rows.work, rows.range, blockIdx.x);
  else
    col_work_body(cols.minmax, n, cols.block_r, cols.t_r, cols.t_c, cols.total_units, cols.work, cols.range,
                  blockIdx.x - blocks_rows);
}

// Unit queues (the tile scheduler).  Workgroup x of a launch runs on XCD x % 8.
// Units are dealt into 8 queues (one per XCD: by slice (batch row, head) when the
// slice count is a multiple of 8, so that the units sharing one head's K/V also
// share one L2), each queue is sorted heaviest first within groups of slices (see
// order_kernel; work quantised to 512 levels), and the queues are interleaved:
// slot 8*s + g = position s of queue g.  The workgroups that run from the start have
// their ticket in their number, later ones draw the next of their XCD's queue when they
// start, so every queue is worked off longest-job-first.  A launch of more units than run
// at once holds more workgroups than tickets, and a workgroup that finds its own queue
// empty draws from the queue that has most left.  (The XCDs do not run at the same
// speed: with equal shares the slowest one finishes about a tenth later than the
// fastest.)
// A slot is the record {unit, first live block, one past the last live block, 0},
// so a workgroup learns all it needs to start from one 16-byte load; slots with
// no unit hold unit = -1.  The kernel also zeroes the 8 queue counters behind
// the slots.
constexpr int kLevels = 512;
constexpr int kGroups = FM_QUEUES;
// Queue of block i of slice s (slices = batch rows x heads, numbered batch-major).  Slices go to
// queues whole, slice s to queue s % 8, as long as they fill rounds of 8; the r < 8 slices left over
// (all slices if there are fewer than 8) are shared block by block: four of them between 2 queues
// each, two between 4 queues each, one between all 8 (r = 4a + 2b + c), which keeps the queues
// equally long and every slice in as few L2s as that allows.
__host__ __device__ inline int fm_queue_of(int s, int i, int whole, int r) {
  if (s < whole) return s % FM_QUEUES;
  int j = s - whole;
  if (r & 4) {
    if (j < 4) return 2 * j + (i & 1);
    j -= 4;
  }
  if (r & 2) {
    if (j < 2) return 4 * j + (i & 3);
    j -= 2;
  }
  return i & 7;
}
// work and range are indexed [batch row][block]; a unit is (batch row, head, block).
// A queue holds its whole slices in groups of FM_QUEUE_CHUNK, one group after the other, and the
// shared slices last: the units that run at the same time then belong to few slices and share their
// K/V (or Q/dO) in the XCD's L2 and in the memory-side cache.  (Ranking a queue's units of ALL slices
// by work alone spreads the resident workgroups over as many slices as the queue has; with 64 slices
// per queue the loops then stream from HBM and lose a quarter of their rate.)  One workgroup of the
// launch sorts one group of one queue.  Within a group units are ranked as rank_of() describes.
struct OrderJob {
  const int* work;
  const int* range;
  int batch, heads, units_per_bh;   // a queue slice: (batch row, head); with grouped K/V heads `heads` counts K/V
                                    // heads and a slice holds the units of all query heads of the group
  int blocks;                       // blocks per (batch row, query head): units_per_bh = group size x blocks
  int max_work, slots;
  i32x4* order;
  int* counters;
};
// Workgroup `block` of `blocks` = 8 x (groups of whole slices + 1): block % 8 is the queue, block / 8 the
// group; the last group is the shared slices, whose workgroups also clear their queue's unused slots
// and counter.
// `unit_work(u)` is {live blocks, first live block, one past the last} of unit u.
template <class UnitWork>
__device__ __forceinline__ void order_body(const OrderJob& job, int block, int blocks, const UnitWork& unit_work) {
  const int heads = job.heads, units_per_bh = job.units_per_bh, max_work = job.max_work;
  const int slots = job.slots;
  i32x4* __restrict__ order = job.order;
  __shared__ int hist[kLevels];
  __shared__ int wave_sum[16];
  const int tid = threadIdx.x;
  const int slices = job.batch * heads;
  const int whole = (slices / kGroups) * kGroups, left = slices - whole;
  const int g = block % kGroups, grp = block / kGroups;
  const bool tail = grp == blocks / kGroups - 1;
  constexpr int chunk = FM_QUEUE_CHUNK;
  // Candidates of this workgroup: the units of its queue's whole slices of the group (slice numbers
  // (grp * chunk + c) * 8 + g), or every unit of the shared slices, of which it keeps its queue's.
  const int first_slice = tail ? whole : (grp * chunk) * kGroups + g;
  const int n_slices = tail ? left : min(chunk, (whole - first_slice + kGroups - 1) / kGroups);
  const int candidates = n_slices * units_per_bh;
  const int pos_base = tail ? (whole / kGroups) * units_per_bh : grp * chunk * units_per_bh;
  auto unit_at = [&](int idx) {   // unit number of candidate idx, or -1 if it belongs to another queue
    const int c = idx / units_per_bh, i = idx - c * units_per_bh;
    const int slice = tail ? first_slice + c : first_slice + c * kGroups;
    if (tail && fm_queue_of(slice, i, whole, left) != g) return -1;
    return slice * units_per_bh + i;
  };
  if (tid < kLevels) hist[tid] = 0;
  if (tail) {
    // this queue's positions behind the whole slices: filled below as far as there are shared slices
    for (int p = pos_base + tid; p * kGroups + g < slots; p += 1024) order[p * kGroups + g] = i32x4{-1, 0, 0, 0};
    if (tid == 0) job.counters[g] = 0;
  }
  __syncthreads();
  auto rank_of = [&](const i32x4& uw) {
    const int w_u = uw[0], mw = max_work > 0 ? max_work : 1;
    // Heavy units (an eighth of the largest possible work or more) are ranked finely by work: their
    // order decides how evenly the queue ends.  Lighter ones are ranked by octave of work and, within
    // an octave, by where their live range starts: units of similar size that stream the same blocks
    // (the rows of one document) then sit next to each other in the queue, run at the same time and
    // share the blocks in L2.
    constexpr int kFine = 384, kOct = 8, kPos = (kLevels - kFine) / kOct;
    int rank;
    const float share = (float)w_u / (float)mw;   // of the largest possible work
    if (share >= 0.125f) {
      rank = min(max((int)((1.f - share) * (8.f / 7.f * (kFine - 1))), 0), kFine - 1);
    } else {
      const int oct = min(max((int)__log2f((float)mw / (8.f * (float)max(w_u, 1))), 0), kOct - 1);
      const int pos = min((int)((float)uw[1] / (float)mw * kPos), kPos - 1);
      rank = kFine + oct * kPos + pos;
    }
    return rank;
  };
  // a thread's first candidate keeps its rank and record between the two passes
  const int u_0 = tid < candidates ? unit_at(tid) : -1;
  i32x4 uw_0 = {0, 0, 0, 0};
  int rank_0 = 0;
  if (u_0 >= 0) {
    uw_0 = unit_work(u_0);
    rank_0 = rank_of(uw_0);
    atomicAdd(&hist[rank_0], 1);
  }
  for (int idx = tid + 1024; idx < candidates; idx += 1024) {
    const int u = unit_at(idx);
    if (u >= 0) atomicAdd(&hist[rank_of(unit_work(u))], 1);
  }
  __syncthreads();
  // exclusive scan of hist (512 entries, one per thread of the first 8 waves)
  const int v = tid < kLevels ? hist[tid] : 0;
  int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(incl, off, 64);
    if ((tid & 63) >= off) incl += y;
  }
  if ((tid & 63) == 63) wave_sum[tid >> 6] = incl;
  __syncthreads();
  int base = 0;
  for (int w = 0; w < (tid >> 6); ++w) base += wave_sum[w];
  __syncthreads();
  if (tid < kLevels) hist[tid] = base + incl - v;   // first queue position (within the group) of this rank
  __syncthreads();
  auto place = [&](int u, int rank, const i32x4& uw) {
    const int slot = (pos_base + atomicAdd(&hist[rank], 1)) * kGroups + g;
    if (slot < slots) order[slot] = i32x4{u, uw[1], uw[2], 0};
  };
  if (u_0 >= 0) place(u_0, rank_0, uw_0);
  for (int idx = tid + 1024; idx < candidates; idx += 1024) {
    const int u = unit_at(idx);
    if (u < 0) continue;
    const i32x4 uw = unit_work(u);
    place(u, rank_of(uw), uw);
  }
}
// Work and live range from the arrays of the work pre-pass.
struct WorkArrays {
  const int* __restrict__ work;
  const int* __restrict__ range;
  int units_per_row, blocks;   // units of a batch row, blocks of a (batch row, query head)
  __device__ __forceinline__ i32x4 operator()(int u) const {
    const int ru = (u / units_per_row) * blocks + u % blocks;
    return i32x4{work[ru], range[2 * ru], range[2 * ru + 1], 0};
  }
};
__device__ __forceinline__ void order_from_arrays(const OrderJob& job, int block, int blocks) {
  order_body(job, block, blocks, WorkArrays{job.work, job.range, job.heads * job.units_per_bh, job.blocks});
}

__global__ __launch_bounds__(1024) void order_kernel(OrderJob job) { order_from_arrays(job, blockIdx.x, gridDim.x); }

// the queues of two passes in one launch: workgroups [0, blocks_a) build job a's, the rest job b's
__global__ __launch_bounds__(1024) void order2_kernel(OrderJob a, int blocks_a, OrderJob b) {
  if ((int)blockIdx.x < blocks_a)
    order_from_arrays(a, blockIdx.x, blocks_a);
  else
    order_from_arrays(b, blockIdx.x - blocks_a, gridDim.x - blocks_a);
}

// The whole setup of a pass (or of the backward's two) in one launch, for sequences of at most FM_ONE_LAUNCH_LENGTH and
// few slices (fm_setup_launches): every queue-building workgroup forms the table and the work of its slices' batch rows
// itself, in LDS, from the bound vectors.  At these lengths that is one 16-byte load per thread and vector and at most
// 32 x 64 tile classes, while each launch of the three-launch form (tables, work, queues) is bound by its start and one
// round trip to memory.
struct SetupJob {
  OrderJob order;          // work and range are not used
  int block_r, block_c;
  int t_r, t_c;
  int cols;                // units are key blocks (else row blocks)
  FmPads pads;
  int* minmax;             // [batch][8][t_c], written for the tile loops
};
struct SetupArgs {
  const int* vec[4];       // LTS, LTE, UTS, UTE: [batch][n]
  int n, np;
  int blocks_first;        // workgroups of job[0], the rest are job[1]'s
  SetupJob job[2];
};
__global__ __launch_bounds__(1024) void setup_kernel(SetupArgs a) {
  constexpr int kMaxTiles = FM_ONE_LAUNCH_LENGTH / 64, kMaxUnits = FM_ONE_LAUNCH_LENGTH / 128, kMaxRows = FM_QUEUES - 1;
  __shared__ i32x4 block_full[kMaxTiles];    // of a key block: LTS max, LTE min, UTS max, UTE min (what T_FULLY asks for)
  __shared__ int work[kMaxRows * kMaxUnits], first[kMaxRows * kMaxUnits], last[kMaxRows * kMaxUnits];
  const bool second = (int)blockIdx.x >= a.blocks_first;
  const SetupJob& job = a.job[second ? 1 : 0];
  const int block = second ? blockIdx.x - a.blocks_first : blockIdx.x;
  const int blocks = second ? gridDim.x - a.blocks_first : a.blocks_first;
  const int n = a.n, t_r = job.t_r, t_c = job.t_c, block_r = job.block_r, units = job.cols ? t_c : t_r;
  const int tid = threadIdx.x;

  // The batch rows of this workgroup's slices (see order_body): two slices 8 apart, or the slices left over.
  const int heads = job.order.heads, slices = job.order.batch * heads;
  const int whole = slices / kGroups * kGroups, g = block % kGroups, grp = block / kGroups;
  const bool tail = grp == blocks / kGroups - 1;
  const int s0 = tail ? whole : grp * FM_QUEUE_CHUNK * kGroups + g;
  const int s1 = tail ? slices - 1 : min(s0 + (FM_QUEUE_CHUNK - 1) * kGroups, whole - kGroups + g);
  const int row0 = s0 / heads, row1 = s1 / heads;                 // s1 < s0: no slice
  const int n_rows = s1 < s0 ? 0 : tail ? row1 - row0 + 1 : (row1 > row0 ? 2 : 1);
  static_assert(FM_QUEUE_CHUNK == 2, "at most two batch rows besides the slices left over");

  for (int i = tid; i < n_rows * kMaxUnits; i += 1024) {
    work[i] = last[i] = 0;
    first[i] = INT32_MAX;
  }
  // a unit's blocks are shared by 1024 / units_p2 threads, which lie units_p2 apart
  int shift = 0;
  while ((1 << shift) < units) ++shift;
  const int my_unit = tid & ((1 << shift) - 1), seg = tid >> shift, segs = 1024 >> shift;
  for (int r = 0; r < n_rows; ++r) {
    const int b = tail ? row0 + r : (r ? row1 : row0);
    // the table goes to memory from the workgroup of the batch row's first slice (of queue 0 if it is shared)
    int* const out = (tail ? g == 0 && b * heads >= whole : b * heads == (r ? s1 : s0)) ? job.minmax + (size_t)b * 8 * t_c
                                                                                        : nullptr;
    // block_c / 4 lanes take a key block, four columns each
    static_assert(FM_ONE_LAUNCH_LENGTH == 4 * 1024, "four columns per thread");
    const int lanes = job.block_c / 4, j = tid / lanes, key = tid * 4;
    i32x4 x[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int* vec = a.vec[v] + (size_t)b * n;
      if (n == a.np) {
        x[v] = *(const i32x4*)(vec + min(key, n - 4));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int y = vec[min(key + e, n - 1)];
          x[v][e] = key + e < n ? y : pad_value(job.pads, v, y);
        }
      }
    }
    int mm[8];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      mm[2 * v] = row16_max(max(max(x[v][0], x[v][1]), max(x[v][2], x[v][3])));
      mm[2 * v + 1] = row16_min(min(min(x[v][0], x[v][1]), min(x[v][2], x[v][3])));
      if (lanes == 32) {
        mm[2 * v] = max(mm[2 * v], __shfl_xor(mm[2 * v], 16, 64));
        mm[2 * v + 1] = min(mm[2 * v + 1], __shfl_xor(mm[2 * v + 1], 16, 64));
      }
    }
    if ((tid & (lanes - 1)) == 0 && j < t_c) {
      block_full[j] = i32x4{mm[LTS_MAX], mm[LTE_MIN], mm[UTS_MAX], mm[UTE_MIN]};
      if (out) {
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e * t_c + j] = mm[e];
      }
    }
    __syncthreads();
    // work and live range of every unit
    const int others = job.cols ? t_r : t_c;
    int cnt = 0, lo = INT32_MAX, hi = 0;
    if (my_unit < units) {
      for (int o = seg; o < others; o += segs) {
        const i32x4 f = block_full[job.cols ? my_unit : o];
        const int r0 = (job.cols ? o : my_unit) * block_r, r1 = min(r0 + block_r, n);
        if (!((r0 >= f[0] && r1 <= f[1]) || (r0 >= f[2] && r1 <= f[3]))) {
          ++cnt;
          lo = min(lo, o);
          hi = o + 1;
        }
      }
      if (cnt) {
        atomicAdd(&work[r * kMaxUnits + my_unit], cnt);
        atomicMin(&first[r * kMaxUnits + my_unit], lo);
        atomicMax(&last[r * kMaxUnits + my_unit], hi);
      }
    }
    __syncthreads();   // the blocks are rebuilt for the next batch row
  }
  const int units_per_row = heads * job.order.units_per_bh, blocks_per_head = job.order.blocks;
  order_body(job.order, block, blocks, [&](int u) {
    const int b = u / units_per_row, i = (tail ? b - row0 : (b > row0 ? 1 : 0)) * kMaxUnits + u % blocks_per_head;
    return i32x4{work[i], work[i] ? first[i] : 0, last[i], 0};
  });
}

}  // namespace fm

using namespace fm;

hipError_t fm_launch_preprocess(const int* lts, const int* lte, const int* uts, const int* ute, int B, int N, int Np,
                                int block_c, FmPads pads, int* minmax, hipStream_t stream) {
  const int t_c = (Np + block_c - 1) / block_c;
  const int total = B * t_c;
  hipLaunchKernelGGL(preprocess_kernel, dim3((total + 3) / 4), dim3(256), 0, stream, lts, lte, uts, ute, N, pads,
                     block_c, t_c, total, minmax);
  return hipGetLastError();
}

hipError_t fm_launch_classify(const int* minmax, int B, int N, int block_r, int block_c, uint8_t* cls,
                              hipStream_t stream) {
  const int t_c = (N + block_c - 1) / block_c;
  const int t_r = (N + block_r - 1) / block_r;
  hipLaunchKernelGGL(classify_kernel, dim3((t_c + 255) / 256, t_r, B), dim3(256), 0, stream, minmax, N, block_r, t_r,
                     t_c, cls);
  return hipGetLastError();
}

// H heads per batch row in groups of `group` that share a K/V head (1: no sharing): the heads of a group
// form one queue slice, so that they run on the XCD whose L2 holds their K/V.
static OrderJob order_job(int* work, int* range, int B, int H, int group, int blocks, int max_work, int* order) {
  const int slots = fm_order_slots(B * H * blocks);
  return OrderJob{work, range, B, H / group, group * blocks, blocks, max_work, slots, (i32x4*)order,
                  order + 4 * (size_t)slots};
}

static WorkJob work_job(const FmSetup& p, int B, int N, int Np, bool cols) {
  const int t_r = (N + p.block_r - 1) / p.block_r, t_c = (Np + p.block_c - 1) / p.block_c;
  return WorkJob{p.minmax, p.block_r, t_r, t_c, B * (cols ? t_c : t_r), p.work, p.range};
}
static OrderJob pass_order_job(const FmSetup& p, const WorkJob& w, int B, int H, int Hk, bool cols) {
  return cols ? order_job(p.work, p.range, B, Hk, 1, w.t_c, w.t_r, p.order)
              : order_job(p.work, p.range, B, H, H / Hk, w.t_r, w.t_c, p.order);
}
static SetupJob setup_job(const FmSetup& p, int B, int H, int Hk, int N, int Np, bool cols) {
  const WorkJob w = work_job(p, B, N, Np, cols);
  return SetupJob{pass_order_job(p, w, B, H, Hk, cols), p.block_r, p.block_c, w.t_r, w.t_c, cols, p.pads, p.minmax};
}

hipError_t fm_launch_setup(const int* lts, const int* lte, const int* uts, const int* ute, int B, int H, int Hk, int N,
                           int Np, const FmSetup& pass, bool cols, hipStream_t stream) {
  const int grid = fm_order_grid(B, Hk);
  if (fm_setup_launches(1, B, Hk, Np, fm_compute_units()) == 1) {
    SetupArgs a{{lts, lte, uts, ute}, N, Np, grid, {setup_job(pass, B, H, Hk, N, Np, cols), {}}};
    hipLaunchKernelGGL(setup_kernel, dim3(grid), dim3(1024), 0, stream, a);
    return hipGetLastError();
  }
  if (hipError_t e = fm_launch_preprocess(lts, lte, uts, ute, B, N, Np, pass.block_c, pass.pads, pass.minmax, stream); e != hipSuccess)
    return e;
  const WorkJob w = work_job(pass, B, N, Np, cols);
  const int work_grid = (w.total_units + 3) / 4;
  if (cols)
    hipLaunchKernelGGL(col_work_kernel, dim3(work_grid), dim3(256), 0, stream, w.minmax, N, w.block_r, w.t_r, w.t_c,
                       w.total_units, w.work, w.range);
  else
    hipLaunchKernelGGL(row_work_kernel, dim3(work_grid), dim3(256), 0, stream, w.minmax, N, w.block_r, w.t_r, w.t_c,
                       w.total_units, w.work, w.range);
  hipLaunchKernelGGL(order_kernel, dim3(grid), dim3(1024), 0, stream, pass_order_job(pass, w, B, H, Hk, cols));
  return hipGetLastError();
}

// The backward's setup: one launch, or three (both min/max tables, both work pre-passes, both passes' queues).
hipError_t fm_launch_bwd_setup(const int* lts, const int* lte, const int* uts, const int* ute, int B, int H, int Hk,
                               int N, int Np, const FmSetup& rows, const FmSetup& cols, hipStream_t stream) {
  const int grid = fm_order_grid(B, Hk);
  if (fm_setup_launches(2, B, Hk, Np, fm_compute_units()) == 1) {
    SetupArgs a{{lts, lte, uts, ute}, N, Np, grid,
                {setup_job(rows, B, H, Hk, N, Np, false), setup_job(cols, B, H, Hk, N, Np, true)}};
    hipLaunchKernelGGL(setup_kernel, dim3(2 * grid), dim3(1024), 0, stream, a);
    return hipGetLastError();
  }
  const WorkJob wr = work_job(rows, B, N, Np, false), wc = work_job(cols, B, N, Np, true);
  const int pre_a = (B * wr.t_c + 3) / 4, pre_b = (B * wc.t_c + 3) / 4;
  hipLaunchKernelGGL(preprocess2_kernel, dim3(pre_a + pre_b), dim3(256), 0, stream, lts, lte, uts, ute, N, Np, B,
                     rows.block_c, rows.pads, rows.minmax, pre_a, cols.block_c, cols.pads, cols.minmax);
  const int work_a = (wr.total_units + 3) / 4, work_b = (wc.total_units + 3) / 4;
  hipLaunchKernelGGL(work2_kernel, dim3(work_a + work_b), dim3(256), 0, stream, wr, work_a, wc, N);
  hipLaunchKernelGGL(order2_kernel, dim3(2 * grid), dim3(1024), 0, stream, pass_order_job(rows, wr, B, H, Hk, false), grid,
                     pass_order_job(cols, wc, B, H, Hk, true));
  return hipGetLastError();
}
