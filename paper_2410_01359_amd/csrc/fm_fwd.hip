// Forward tile loop (Algorithm 1) for gfx950.
//
// One workgroup (4 waves) per (batch, head, block of 128 query rows).  Each wave
// owns 32 query rows for the whole kernel and walks the key blocks that the
// min/max tables do not prove fully masked.  Scores are computed transposed,
// S^T = K Q^T, so that after the MFMA every lane holds ONE query column: row
// max / row sum are per-lane loops plus one exchange with the lane 32 away, the
// running rescale of O is a per-lane scalar, and P^T is already in the
// B-operand layout of the second product O^T += V^T P^T.  K tiles are read
// from LDS as A operands (128-bit reads), V tiles through the LDS transpose
// read.  Q stays in registers.
//
// The loop is software-pipelined over key tiles: while the exp / row-sum
// arithmetic of tile t runs on the vector unit, the matrix unit already computes
// the scores of tile t+1 into a second accumulator set, so a wave keeps both
// units busy by itself instead of relying on the other resident wave being in
// the complementary phase.  K and V therefore travel in separate two-deep LDS
// rings: iteration t reads K(t+1) and V(t) while K(t+2) and V(t+1) are in flight.
#include "fm_common.h"
#include "fm_kernels.h"

namespace fm {

#ifndef FM_FWD_EXP_A
#define FM_FWD_EXP_A 20
#endif

// S: groups of waves that share a unit's key tiles, each tile of the list belongs to one group (2: direct units only).
// WR: waves of a group, 32 query rows each.
template <int D, int S = 1, int WR = 4>
struct FwdCfg {
  static constexpr int KT = FM_FWD_BC;          // keys per tile
  static constexpr int BR = 32 * WR;            // query rows per workgroup
  static constexpr int THREADS = 64 * S * WR;
  using L = TileLayout<D>;
  static constexpr int K_BYTES = KT * L::RS;
  static constexpr int V_BYTES = KT * L::RS;
  static constexpr int BND_BYTES = 4 * KT * 4;  // LTS, LTE, UTS, UTE slices of one tile, kept behind its V tile
  static constexpr int VSTAGE = V_BYTES + BND_BYTES;
  static constexpr int LIST_CAP = 1024;         // key blocks classified per pass
  static constexpr int LIST_OFF = 0;
  static constexpr int CNT_OFF = LIST_CAP * 4;
  static constexpr int K_OFF = CNT_OFF + 64;
  static constexpr int V_OFF = K_OFF + 2 * S * K_BYTES;   // two stages of S tiles each
  static constexpr int LDS_BYTES = V_OFF + 2 * S * VSTAGE;
  static constexpr int PER_CU = fm_fwd_per_cu(D);         // workgroups of 128-row units on a compute unit
};

// Per-wave constants of the tile loop.
template <int D>
struct FwdWave {
  int a_off;               // operand rows: row c, bytes 16 g (slice kk adds 32 kk through TileLayout::add_col)
  int t_off[2];            // transpose reads: row 4 g + i16/4 (+8), bytes 32 half + 8 (i16 & 3) (d block db adds 64 db)
  int row;                 // this lane's query row
  int g;
  float sc;                // scale * log2(e)
};

// Softmax state of a lane's query: P = exp2(scale log2(e) S + neg_ref).
constexpr float kRescaleGap = 8.f;
struct FwdSoftmax {
  float neg_ref;   // minus the reference maximum (log2 domain), 0 before the first finite one
  float limit;     // the reference moves when a tile's maximum exceeds this: reference + gap, -inf before the first finite one
  float l;         // sum of P over this lane's keys
  __device__ __forceinline__ float reference() const { return limit == -INFINITY ? -INFINITY : -neg_ref; }
};

// One pipeline step: exp / row-sum arithmetic and O^T += V^T P^T of the tile whose raw scores
// are in `cur` (masked first if `masked` != 0), and the raw scores of the NEXT tile (K tile at
// k_next) into `nxt`.
template <int D>
__device__ __forceinline__ void fwd_step(f32x16 (&cur)[2], f32x16 (&nxt)[2], f32x16 (&oacc)[D / 32],
                                         const bf16x8 (&qreg)[D / 16], FwdSoftmax& sm,
                                         const char* k_next, const char* vs, const int* bnd, int masked,
                                         const FwdWave<D>& w) {
  using C = FwdCfg<D>;
  constexpr int KT = C::KT, NKB = KT / 32, NDB = D / 32, NKK = D / 16;
  static_assert(NKB == 2, "two 32-key blocks per tile");
  // per-lane LDS offsets, made opaque once per tile so that what is derived from them is
  // recomputed (one vector op each) instead of being hoisted out of the tile loop into registers
  const int a_b = opaque(w.a_off), t_b0 = opaque(w.t_off[0]), t_b1 = opaque(w.t_off[1]);

  if (masked) {
    const int* bnd_g = (const int*)((const char*)bnd + opaque(16 * w.g));
    // A sub-tile that Equation 4 proves fully masked for this wave takes the same path and ends
    // with every score at -inf.  `masked` says which pairs the workgroup's tile needs (1 = LT,
    // 2 = UT, 3 = both; 5, 6, 7 = the same with a single comparison per pair, see entry_mask_mode):
    // a pair that is not needed masks no element of the tile, so leaving it
    // out is exact -- and most partially masked tiles (a causal diagonal, a window edge, a
    // document boundary) need only one.
    // The bounds of GROUPS groups of four keys are fetched together, into the registers that the next tile's scores take
    // later: one group at a time, a masked tile waited for LDS eight times in a row.  With the single comparisons of mode
    // 7, where both pairs took two each: forward, documents, d = 128 N = 1000 23.4 -> 21.7 us, N = 4099 89.8 -> 84.6,
    // d = 64 N = 8192 170.9 -> 157.7, window 256 at N = 32768 134.8 -> 126.0.
    auto bounds = [&](int which, int rq8) __attribute__((always_inline)) {   // group rq8 of the tile's 8 of this lane
      return *(const i32x4*)(bnd_g + which * KT + (rq8 / 4) * 32 + 8 * (rq8 % 4));
    };
    if (masked == 3) {
      constexpr int GROUPS = 2;
#pragma unroll
      for (int q0 = 0; q0 < 8; q0 += GROUPS) {
        i32x4 b[GROUPS][4];
#pragma unroll
        for (int q = 0; q < GROUPS; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) b[q][v] = bounds(v, q0 + q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < GROUPS; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool hit = ((w.row >= b[q][0][e]) & (w.row < b[q][1][e])) | ((w.row >= b[q][2][e]) & (w.row < b[q][3][e]));
            if (hit) cur[(q0 + q) / 4][(q0 + q) % 4 * 4 + e] = -INFINITY;
          }
        __builtin_amdgcn_sched_barrier(0);  // keep the bound reads of later steps from piling up in registers
      }
    } else if (masked == 7) {   // both pairs, one comparison each: row >= LTS or row < UTE
      constexpr int GROUPS = 4;
#pragma unroll
      for (int q0 = 0; q0 < 8; q0 += GROUPS) {
        i32x4 b[GROUPS][2];
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) {
          b[q][0] = bounds(0, q0 + q);
          b[q][1] = bounds(3, q0 + q);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < GROUPS; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if ((w.row >= b[q][0][e]) | (w.row < b[q][1][e])) cur[(q0 + q) / 4][(q0 + q) % 4 * 4 + e] = -INFINITY;
        __builtin_amdgcn_sched_barrier(0);
      }
    } else if (masked & 4) {
      // one pair, decided by one comparison per element (5: row >= LTS, 6: row < UTE): one bound per key
      constexpr int GROUPS = 8;
      i32x4 b[GROUPS];
      if (masked == 5) {
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) b[q] = bounds(0, q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) hide4(cur[q / 4], q % 4 * 4, [&](int e) { return w.row >= b[q][e]; });
      } else {
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) b[q] = bounds(3, q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) hide4(cur[q / 4], q % 4 * 4, [&](int e) { return w.row < b[q][e]; });
      }
      __builtin_amdgcn_sched_barrier(0);
    } else {
      constexpr int GROUPS = 4;
      const int lo = masked == 2 ? 2 : 0;   // the one pair that is needed
#pragma unroll
      for (int q0 = 0; q0 < 8; q0 += GROUPS) {
        i32x4 b[GROUPS][2];
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) {
          b[q][0] = bounds(lo, q0 + q);
          b[q][1] = bounds(lo + 1, q0 + q);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < GROUPS; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool hit = (w.row >= b[q][0][e]) & (w.row < b[q][1][e]);
            if (hit) cur[(q0 + q) / 4][(q0 + q) % 4 * 4 + e] = -INFINITY;
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ---- stream A: S^T(next) = K Q^T on the matrix unit, softmax(cur) on the vector unit.
  // MFMA step n: chain kb = n % 2, slice kk = n / 2 (the two accumulation chains alternate);
  // its K operand is fetched about RS steps ahead into a small register ring, two at a time and the later step's first: LDS answers
  // in order, so one wait covers both (15 instead of 29 waits a tile in both streams at d = 128).  Forward, before / now: prefix 4096 of
  // 32768 3920 / 3876 us, skewed documents at 131072 2562 / 2510, shared questions 16300 362 / 358, documents 1000 24.1 / 23.8, 4099
  // at d = 64 59.0 / 59.1.  (In the dQ and dK/dV loops, whose reads fill more of LDS's time, the bursts cost 1 to 4 %.)
  constexpr int NS = NKB * NKK, RS = 4;
  constexpr int NMAX = 4;                          // steps that carry the running max (8 elements each)
  constexpr int NEXP = NS - NMAX - 1;              // steps that carry exponentials
  // The exponentials of the first EXP_A elements (of 32 per lane) ride along with these score
  // MFMAs, the rest with the first half of the second product below (which only needs the first
  // 16): one product's shadow alone is too short for all of them.
  constexpr int EXP_A = FM_FWD_EXP_A;
  constexpr int EPS = (EXP_A + NEXP - 1) / NEXP;   // elements per such step
  bf16x8 kring[RS];
  auto k_operand = [&](int n) __attribute__((always_inline)) {
    return *(const bf16x8*)(k_next + (n % NKB) * 32 * C::L::RS + C::L::add_col(a_b, (n / NKB) * 32));
  };
  const f32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int n = 0; n < RS; ++n) {
    kring[n ^ 1] = k_operand(n ^ 1);
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_sched_barrier(0);
  float mx = -INFINITY, rs = 0.f;
#pragma unroll
  for (int n = 0; n < NS; ++n) {
    nxt[n % NKB] = mfma32(kring[n % RS], qreg[n / NKB], n < NKB ? zero : nxt[n % NKB]);
    if (n % 2 == 1 && n + RS < NS) {
      kring[n % RS] = k_operand(n + RS);
      __builtin_amdgcn_sched_barrier(0);
      kring[(n - 1) % RS] = k_operand(n - 1 + RS);
    }
    if (n < NMAX) {
#pragma unroll
      for (int e = 8 * n; e < 8 * n + 8; ++e) mx = fmaxf(mx, cur[e / 16][e % 16]);
    } else if (n == NMAX) {
      // A lane has the maximum over its half of the query's keys.  Whether any query's reference moves needs no exchange
      // between the two halves: it does where one of them asks for it.  (With the exchange and the reference's sign on every
      // tile's path, ten instructions one behind the other: prefix 32768 at d = 64 4466 -> 4399 us, d = 128 3753 -> 3732.)
      mx *= w.sc;
      if (__any(mx > sm.limit)) {   // also on the first finite maximum
        // The reference maximum only moves when a tile's maximum exceeds it by more than the
        // gap (log2 units), so this rescale of O and l is rare; any reference is a valid one,
        // P just grows up to 2^gap.
        mx = fmaxf(mx, partner32(mx));
        const float m_run = sm.reference(), m_new = mx > sm.limit ? mx : m_run;
        const float alpha = (m_new == -INFINITY) ? 1.f : fast_exp2(m_run - m_new);
        sm.neg_ref = (m_new == -INFINITY) ? 0.f : -m_new;
        sm.limit = m_new + kRescaleGap;
        sm.l *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
      }
    } else {
      const int j = n - NMAX - 1;
#pragma unroll
      for (int e = j * EPS; e < (j + 1) * EPS && e < EXP_A; ++e) {
        const float p = fast_exp2(__builtin_fmaf(cur[e / 16][e % 16], w.sc, sm.neg_ref));
        cur[e / 16][e % 16] = p;
        rs += p;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- stream B: O^T += V^T P^T, step n = (16-key group n / NDB, d block n % NDB)
  constexpr int NP = NKB * 2 * NDB, RP = 4;
  bf16x8 vring[RP];
  auto v_operand = [&](int n) __attribute__((always_inline)) {
    const char* vrow = vs + ((n / NDB) * 16) * C::L::RS;   // group n / NDB = (kb, h): 16 keys each
    return cat4(lds_read_tr16(vrow + C::L::add_col(t_b0, (n % NDB) * 64)),
                lds_read_tr16(vrow + C::L::add_col(t_b1, (n % NDB) * 64)));
  };
#pragma unroll
  for (int n = 0; n < RP; ++n) {
    vring[n ^ 1] = v_operand(n ^ 1);
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < NP; ++n) {
    const int grp = n / NDB, kb = grp / 2, h = grp % 2, db = n % NDB;
    bf16x8 pb;
#pragma unroll
    for (int e = 0; e < 8; ++e) pb[e] = (__bf16)cur[kb][8 * h + e];
    oacc[db] = mfma32(vring[n % RP], pb, oacc[db]);
    if (n % 2 == 1 && n + RP < NP) {
      vring[n % RP] = v_operand(n + RP);
      __builtin_amdgcn_sched_barrier(0);
      vring[(n - 1) % RP] = v_operand(n - 1 + RP);
    }
    if (n < NP / 2) {   // the remaining exponentials (second 32-key block), beside the first block's MFMAs
      constexpr int EPB = (32 - EXP_A + NP / 2 - 1) / (NP / 2);
#pragma unroll
      for (int e = EXP_A + n * EPB; e < EXP_A + (n + 1) * EPB && e < 32; ++e) {
        const float p = fast_exp2(__builtin_fmaf(cur[e / 16][e % 16], w.sc, sm.neg_ref));
        cur[e / 16][e % 16] = p;
        rs += p;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  sm.l += rs;
}

// RAGGED: the sequence length is not a multiple of 128.  The loops then run at the padded length
// Np (tables and lists are built for it; the padding columns are masked for every row), tile copies that reach past row N clamp their source rows, and rows >= N are
// computed but not stored.
// GEN: tensors with caller-given strides and fewer K/V heads than query heads (see FmFwdArgs).
// DIRECT: direct units (see fm_common.h), else queued ones.
template <int D, bool RAGGED, bool GEN, int S, int WR, bool DIRECT>
__device__ __forceinline__ void fwd_body(const FmFwdKernelArgs<GEN>& a) {
  using C = FwdCfg<D, S, WR>;
  // Four waves copy a tile, 16 of its 64 rows each: a group of four its own tiles, a group of two every tile
  // together with the other group.
  constexpr int NT = WR == 4 ? 1 : S;     // tiles per step that a wave takes part in copying
  constexpr int KT = C::KT, NKB = KT / 32, NDB = D / 32, NKK = D / 16;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int t_r = ((RAGGED ? a.N : a.Np) + C::BR - 1) / C::BR;
  i32x4 rec = {-1, 0, 0, 0};
  int bh, i_blk;   // batch row and head, row block
  if (!DIRECT) {
    rec = queue_take(a.queue, (int*)(smem + C::CNT_OFF) + 8);
    if (rec[0] < 0) return;
    bh = rec[0] / t_r;
    i_blk = rec[0] - bh * t_r;
  } else {
    args_at_once(a.order, a.q, a.lts, a.lte, a.uts, a.ute, a.N, a.Np, a.H);
    const FmDirectUnit u = fm_direct_unit<GEN>(a.order, (int)blockIdx.x);
    if (u.block < 0) return;
    bh = GEN ? u.slice * (int)a.order.group.n + u.member : u.slice;
    i_blk = t_r - 1 - u.block;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, c = lane & 31;
  const int N = a.Np, H = a.H;            // padded length: what the loops and tables see
  const int Nr = RAGGED ? a.N : a.Np;     // rows the tensors really have
  const int t_c = N / KT;
  const int j_lo = DIRECT ? 0 : rec[1], j_hi = DIRECT ? t_c : rec[2];
  const int b = bh / H;
  const int q0 = i_blk * C::BR;
  const int wrow = S == 1 ? wave : wave % WR, grp = S == 1 ? 0 : wave / WR;
  const int cwave = S * WR == 4 ? wave : wave % 4;             // which quarter of a tile it copies
  const int sub0 = WR == 4 ? grp : 0;     // first of the NT tiles of a step that it copies
  const int qw0 = q0 + wrow * 32;

  const int h = bh - b * H, hk = GEN ? h / (H / a.Hk) : h, Hk = GEN ? a.Hk : H;
  const __bf16* qp = slice_ptr<D, GEN>(a.q, a.sq, b, h, H, Nr);
  const __bf16* kp = slice_ptr<D, GEN>(a.k, a.sk, b, hk, Hk, Nr);
  const __bf16* vp = slice_ptr<D, GEN>(a.v, a.sv, b, hk, Hk, Nr);
  const int q_rs = row_stride<D, GEN>(a.sq), k_rs = row_stride<D, GEN>(a.sk), v_rs = row_stride<D, GEN>(a.sv);
  const int* table = a.minmax + (size_t)b * 8 * t_c;
  // lanes of wave 0 copy the four bound slices of a partially masked tile: lane l moves
  // 16 bytes of vector l / 16
  const int* my_bvec;
  {
    const int which = lane >> 4;
    const int* p = a.lts;
    if (which == 1) p = a.lte;
    if (which == 2) p = a.uts;
    if (which == 3) p = a.ute;
    my_bvec = p + (size_t)b * Nr + (lane & 15) * 4;
  }
  // RAGGED: rows of the bound vectors are 4-byte aligned only and the last key block reaches past their end:
  // wave w copies one vector's slice, 4 bytes per lane
  const int* wave_bvec = (cwave == 0 ? a.lts : cwave == 1 ? a.lte : cwave == 2 ? a.uts : a.ute) + (size_t)b * Nr;
  CopyLanes<D> copy_lanes, copy_lanes_v_;
  copy_lanes.init(lane, 2 * k_rs);
  if (GEN) copy_lanes_v_.init(lane, 2 * v_rs);
  const CopyLanes<D>& copy_lanes_v = GEN ? copy_lanes_v_ : copy_lanes;
  const char* const kp_wave = CopyLanes<D>::wave_base(kp, cwave, 2 * k_rs);
  const char* const vp_wave = CopyLanes<D>::wave_base(vp, cwave, 2 * v_rs);

  int* list = (int*)(smem + C::LIST_OFF);
  const int* bnd_rows[4] = {a.lts + (size_t)b * Nr, a.lte + (size_t)b * Nr, a.uts + (size_t)b * Nr, a.ute + (size_t)b * Nr};
  // Where one pass covers all key blocks, their bounds are requested ahead of the rows and classified while those are in
  // flight.  With more passes it would be one more round trip: two are requested together then.
  DirectPass<RAGGED, T_UNMASKED, WR, S * WR> first;
  static_assert(first.BLOCKS <= C::LIST_CAP, "a pass fits the list");
  const bool one_pass = DIRECT && t_c <= first.BLOCKS;
  if (one_pass) {
    first.load(bnd_rows, Nr, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  // Q fragments (B operand of S^T = K Q^T): lane holds Q[row c][16 kk + 8 g ..+7].
  bf16x8 qreg[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk)
    qreg[kk] = *(const bf16x8*)(qp + (size_t)(RAGGED ? min(qw0 + c, Nr - 1) : qw0 + c) * q_rs + kk * 16 + 8 * g);
  if (one_pass) {
    __builtin_amdgcn_sched_barrier(0);   // behind the requests for the rows
    first.classify(Nr, 0, 0, t_c, q0, min(q0 + C::BR, Nr), list);
  }

  f32x16 oacc[NDB];
  FwdSoftmax sm = {0.f, -INFINITY, 0.f};
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;

  int* wave_cnt = (int*)(smem + C::CNT_OFF);
  FwdWave<D> w;
  w.sc = a.scale * kLog2e;  // > 0 (checked on the host): scores stay raw, exp2(s*sc - m) is one fma + one exp
  w.row = qw0 + c;
  w.g = g;
  {
    const int i16 = lane & 15, half = (lane >> 4) & 1;
    w.a_off = C::L::off(c, 16 * g);
#pragma unroll
    for (int hi = 0; hi < 2; ++hi) w.t_off[hi] = C::L::off(4 * g + (i16 >> 2) + 8 * hi, (16 * half + 4 * (i16 & 3)) * 2);
  }

  // Asynchronous copies of list entry ENTRY: its K tile into K stage KBUF / its V tile (and, if the
  // workgroup's tile is partially masked, its bound slices) into V stage VBUF.
#define FM_LOAD_K(ENTRY, KBUF, SUB)                                                              \
  {                                                                                              \
    const int j_ = entry_block(ENTRY, chunk);                                                    \
    char* st_ = smem + C::K_OFF + ((KBUF) * S + (SUB)) * C::K_BYTES;                             \
    if (RAGGED && (j_ + 1) * KT > Nr)                                                            \
      tile_load_async_clamped<D>(kp, j_ * KT, Nr, st_, cwave, lane, 2 * k_rs);                    \
    else                                                                                         \
      tile_load_async<D>(kp_wave + (size_t)(2 * j_ * KT) * k_rs, copy_lanes, st_, cwave);         \
  }
#define FM_LOAD_V(ENTRY, VBUF, SUB)                                                              \
  {                                                                                              \
    const int j_ = entry_block(ENTRY, chunk);                                                    \
    char* st_ = smem + C::V_OFF + ((VBUF) * S + (SUB)) * C::VSTAGE;                              \
    if (RAGGED && (j_ + 1) * KT > Nr)                                                            \
      tile_load_async_clamped<D>(vp, j_ * KT, Nr, st_, cwave, lane, 2 * v_rs);                    \
    else                                                                                         \
      tile_load_async<D>(vp_wave + (size_t)(2 * j_ * KT) * v_rs, copy_lanes_v, st_, cwave);       \
    if (entry_tile_class(ENTRY) == T_PARTIAL) {                                                  \
      if (RAGGED)                                                                                \
        async_copy4(bound_or_pad(wave_bvec, cwave, j_ * KT + lane, Nr),                           \
                    lds_address(st_ + C::V_BYTES) + cwave * (KT * 4));                            \
      else if (cwave == 0)                                                                        \
        async_copy16(my_bvec + j_ * KT, lds_address(st_ + C::V_BYTES));                          \
    }                                                                                            \
  }
  // One iteration: step T (tiles S T .. S T + S - 1 of the list, one per group of waves) with scores in CUR, scores
  // of step T + 1 into NXT.  Entries past the end of the list are clamped to the last one: nothing is copied for
  // them, and the scores the last step computes from the stale K stage are never used.  A group without a tile in
  // the last step only takes part in the copies and the barrier.
#define FM_STEP(T, CUR, NXT)                                                                     \
  {                                                                                              \
    /* the list entries that join the window at the next step: read now, picked up behind the */ \
    /* step's barrier, so that no step starts by waiting for LDS                               */ \
    int v_3[NT];                                                                                 \
    _Pragma("unroll") for (int s_ = 0; s_ < NT; ++s_) v_3[s_] = list[min(S * ((T) + 3) + sub0 + s_, n_live - 1)]; \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    _Pragma("unroll") for (int s_ = 0; s_ < NT; ++s_) {                                          \
      if (S * ((T) + 2) + sub0 + s_ < n_live) FM_LOAD_K(e_2[s_], (T) & 1, sub0 + s_);            \
      if (S * ((T) + 1) + sub0 + s_ < n_live) FM_LOAD_V(e_1[s_], ((T) + 1) & 1, sub0 + s_);      \
    }                                                                                            \
    const char* vs_ = smem + C::V_OFF + (((T) & 1) * S + grp) * C::VSTAGE;                       \
    const int e_own = NT == 1 || grp == 0 ? e_t[0] : e_t[NT - 1];                                  \
    if (S == 1 || S * (T) + grp < n_live)                                                        \
      fwd_step<D>(CUR, NXT, oacc, qreg, sm,                                                      \
                  smem + C::K_OFF + ((((T) + 1) & 1) * S + grp) * C::K_BYTES, vs_,               \
                  (const int*)(vs_ + C::V_BYTES),                                                \
                  entry_wave_class(e_own, wrow) != T_UNMASKED ? entry_mask_mode(e_own) : 0, w);  \
    async_wait<0>();   /* K(T+2) and V(T+1) have landed ... */                                   \
    barrier_nofence(); /* ... for every wave, and every wave is done with K(T+1) and V(T) */     \
    _Pragma("unroll") for (int s_ = 0; s_ < NT; ++s_) {                                          \
      e_t[s_] = e_1[s_];                                                                         \
      e_1[s_] = e_2[s_];                                                                         \
      e_2[s_] = __builtin_amdgcn_readfirstlane(v_3[s_]);                                         \
    }                                                                                            \
  }

  // only the key blocks [j_lo, j_hi) can be live for this row block (found by the work pre-pass)
  for (int chunk = j_lo; chunk < j_hi; chunk += C::LIST_CAP) {
    const int chunk_end = min(chunk + C::LIST_CAP, j_hi), r1 = min(q0 + C::BR, Nr);
    int n_live;
    if constexpr (!DIRECT) {
      n_live = build_live_key_blocks<T_UNMASKED>(table, t_c, chunk, chunk_end, q0, r1, C::BR / 4, list, wave_cnt);
    } else {
      n_live = build_live_key_blocks_direct<RAGGED, T_UNMASKED, WR, S * WR>(one_pass, bnd_rows, Nr, chunk, chunk_end, q0, r1, list, wave_cnt);
    }
    if (n_live == 0) continue;
    // The Q rows are waited for here, behind the list that their loads were in flight beside.  (No-op after the first pass.)
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) settle(qreg[kk]);
    // the entries of steps T, T + 1, T + 2 of the step about to run (clamped to the last one)
    int e_t[NT], e_1[NT], e_2[NT];
#pragma unroll
    for (int s_ = 0; s_ < NT; ++s_) {
      e_t[s_] = __builtin_amdgcn_readfirstlane(list[min(sub0 + s_, n_live - 1)]);
      e_1[s_] = __builtin_amdgcn_readfirstlane(list[min(S + sub0 + s_, n_live - 1)]);
      e_2[s_] = __builtin_amdgcn_readfirstlane(list[min(2 * S + sub0 + s_, n_live - 1)]);
    }
    {
#pragma unroll
      for (int s_ = 0; s_ < NT; ++s_) FM_LOAD_K(e_t[s_], 0, sub0 + s_);
#pragma unroll
      for (int s_ = 0; s_ < NT; ++s_) {
        FM_LOAD_V(e_t[s_], 0, sub0 + s_);
        FM_LOAD_K(e_1[s_], 1, sub0 + s_);
      }
      // the first scores need the first K tiles only: V and the K after them (at least as many copies) may be in flight
      async_wait<2 * NT * CopyLanes<D>::NINST>();
      barrier_nofence();
    }
    // scores of the first tile
    f32x16 s0[NKB], s1[NKB];
    {
      const char* ks = smem + C::K_OFF + grp * C::K_BYTES;
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s0[kb][r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
          s0[kb] = mfma32(*(const bf16x8*)(ks + kb * 32 * C::L::RS + C::L::add_col(w.a_off, kk * 32)), qreg[kk], s0[kb]);
      async_wait<0>();
      barrier_nofence();   // the first iteration refills this K stage: every wave must have read it
    }
    const int n_steps = (n_live + S - 1) / S;
    for (int t = 0; t < n_steps; t += 2) {
      FM_STEP(t, s0, s1)
      if (t + 1 < n_steps) FM_STEP(t + 1, s1, s0)
    }
    __syncthreads();     // the list is rebuilt by the next pass
  }
#undef FM_STEP
#undef FM_LOAD_K
#undef FM_LOAD_V

  // epilogue: O / l, lse = m + log(l)   (m, l in the log2 domain)
  __bf16* op = (__bf16*)slice_ptr<D, GEN>(a.out, a.so, b, h, H, Nr);
  const int o_rs = row_stride<D, GEN>(a.so);
  float* lp = a.lse + (size_t)bh * Nr;
  {
    if (S == 2) {
      // The two groups' softmax states of the same rows meet in LDS (nothing is in flight into the stages, every
      // wave is past its last tile): the second group leaves m, l and O of its rows, the first one brings both to
      // the larger reference maximum and adds.
      static_assert(S == 1 || WR * 64 * (16 * NDB + 2) * 4 + 4 * RowStage<D>::BYTES <= C::LDS_BYTES - C::K_OFF, "exchange fits the stages");
      float* const part = (float*)(smem + C::K_OFF + 4 * RowStage<D>::BYTES) + wrow * 64 * (16 * NDB + 2) + lane * 4;
      float* const part_ml = (float*)(smem + C::K_OFF + 4 * RowStage<D>::BYTES) + wrow * 64 * (16 * NDB + 2) + 64 * 16 * NDB + lane;
      if (grp == 1) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int rq = 0; rq < 4; ++rq)
            *(f32x4*)(part + (db * 4 + rq) * 256) =
                f32x4{oacc[db][rq * 4], oacc[db][rq * 4 + 1], oacc[db][rq * 4 + 2], oacc[db][rq * 4 + 3]};
        part_ml[0] = sm.reference();
        part_ml[64] = sm.l;
      }
      barrier_nofence();
      if (grp == 1) return;
      const float m_0 = sm.reference(), m_1 = part_ml[0], m_new = fmaxf(m_0, m_1);
      const float a_0 = m_0 == -INFINITY ? 0.f : fast_exp2(m_0 - m_new);
      const float a_1 = m_1 == -INFINITY ? 0.f : fast_exp2(m_1 - m_new);
      sm.l = sm.l * a_0 + part_ml[64] * a_1;
      sm.neg_ref = -m_new;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          const f32x4 o = *(const f32x4*)(part + (db * 4 + rq) * 256);
#pragma unroll
          for (int e = 0; e < 4; ++e) oacc[db][rq * 4 + e] = oacc[db][rq * 4 + e] * a_0 + o[e] * a_1;
        }
    }
    const float lt = sm.l + partner32(sm.l);
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    const int row = qw0 + c;
    // every wave is past its last tile and nothing is in flight into the K / V stages (the barrier that
    // ends a pass over the list): their first bytes serve as the waves' store staging
    using RSt = RowStage<D>;
    static_assert(4 * RSt::BYTES <= C::LDS_BYTES - C::K_OFF, "store staging fits the K / V stages");
    char* stage = smem + C::K_OFF + wave * RSt::BYTES;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(oacc[db][rq * 4 + e] * inv);
        RSt::put(stage, c, g, db, rq, o4);
      }
    RSt::flush(stage, op + (size_t)qw0 * o_rs, o_rs, lane, RAGGED ? min(32, Nr - qw0) : 32);
    if ((!RAGGED || row < Nr) && g == 0) lp[row] = lt > 0.f ? (fast_log2(lt) - sm.neg_ref) * kLn2 : -INFINITY;
  }
}

template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(256, FwdCfg<D>::PER_CU) void fwd_kernel(FmFwdKernelArgs<GEN> a) {
  fwd_body<D, RAGGED, GEN, 1, 4, false>(a);
}
// Direct units.  LDS for two tiles per step leaves one workgroup per compute unit at d = 128, two at d = 64.
template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(256, FwdCfg<D>::PER_CU) void single_fwd_kernel(FmFwdKernelArgs<GEN> a) {
  fwd_body<D, RAGGED, GEN, 1, 4, true>(a);
}
template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void direct_fwd_kernel(FmFwdKernelArgs<GEN> a) {
  fwd_body<D, RAGGED, GEN, 2, 2, true>(a);
}
template <int D, bool RAGGED, bool GEN>
__global__ __launch_bounds__(512, 1) void wide_fwd_kernel(FmFwdKernelArgs<GEN> a) {
  fwd_body<D, RAGGED, GEN, 2, 4, true>(a);
}

}  // namespace fm

using namespace fm;

template <int D, bool RAGGED, bool GEN, FmUnits U>
struct FwdLaunch {
  using C = FwdCfg<D, fm_groups(U), fm_group_waves(U)>;
  static constexpr auto kernel() {
    if constexpr (U == FM_QUEUED) return fwd_kernel<D, RAGGED, GEN>;
    else if constexpr (U == FM_DIRECT) return single_fwd_kernel<D, RAGGED, GEN>;
    else if constexpr (U == FM_DIRECT_HALVED) return direct_fwd_kernel<D, RAGGED, GEN>;
    else return wide_fwd_kernel<D, RAGGED, GEN>;
  }
  static FmLdsLimit lds() { return {(const void*)kernel(), C::LDS_BYTES}; }
};

template <int D, bool RAGGED, bool GEN, FmUnits U>
static hipError_t launch_fwd_s(const FmFwdArgs& a, hipStream_t stream) {
  using L = FwdLaunch<D, RAGGED, GEN, U>;
  using C = typename L::C;
  auto args = fm_kernel_args<GEN>(a);
  const int blocks = (a.N + C::BR - 1) / C::BR;
  if (U == FM_QUEUED) args.queue = fm_queue_for_launch(a.queue, FwdCfg<D>::PER_CU);
  else args.order = fm_direct_order(a.B * a.Hk, a.H / a.Hk, blocks, a.B * a.H * blocks <= fm_compute_units());
  const int grid = U == FM_QUEUED ? fm_launch_grid(args.queue) : fm_direct_grid(args.order);
  hipLaunchKernelGGL(L::kernel(), dim3(grid), dim3(C::THREADS), C::LDS_BYTES, stream, args);
  return hipGetLastError();
}

template <int D, bool RAGGED, bool GEN>
static hipError_t launch_fwd_t(const FmFwdArgs& a, hipStream_t stream) {
  static bool allowed[FM_MAX_DEVICES] = {};
  if (hipError_t e = fm_allow_lds({FwdLaunch<D, RAGGED, GEN, FM_QUEUED>::lds(),
                                   FwdLaunch<D, RAGGED, GEN, FM_DIRECT>::lds(),
                                   FwdLaunch<D, RAGGED, GEN, FM_DIRECT_HALVED>::lds(),
                                   FwdLaunch<D, RAGGED, GEN, D == 128 ? FM_DIRECT_PAIRED : FM_QUEUED>::lds()},
                                  allowed);
      e != hipSuccess)
    return e;
  switch (a.units) {
    case FM_DIRECT: return launch_fwd_s<D, RAGGED, GEN, FM_DIRECT>(a, stream);
    case FM_DIRECT_HALVED: return launch_fwd_s<D, RAGGED, GEN, FM_DIRECT_HALVED>(a, stream);
    case FM_DIRECT_PAIRED:
      if constexpr (D == 128) return launch_fwd_s<D, RAGGED, GEN, FM_DIRECT_PAIRED>(a, stream);
    default: return launch_fwd_s<D, RAGGED, GEN, FM_QUEUED>(a, stream);
  }
}

template <int D>
static hipError_t launch_fwd_d(const FmFwdArgs& a, hipStream_t stream) {
  const bool ragged = a.Np != a.N;
  if (a.general) return ragged ? launch_fwd_t<D, true, true>(a, stream) : launch_fwd_t<D, false, true>(a, stream);
  return ragged ? launch_fwd_t<D, true, false>(a, stream) : launch_fwd_t<D, false, false>(a, stream);
}

hipError_t fm_launch_fwd(const FmFwdArgs& a, hipStream_t stream) {
  static_assert(FM_FWD_BR == FwdCfg<128>::BR, "forward row block");
  return a.d == 128 ? launch_fwd_d<128>(a, stream) : launch_fwd_d<64>(a, stream);
}
